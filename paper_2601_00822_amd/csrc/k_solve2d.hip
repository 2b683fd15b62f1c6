// Whole basic-scheme iterations of small 2D solves, one workgroup per solve.
//
// The launches of a 2D iteration (x pass, outer pass, reduction) take 4 to 9 us
// each for a 64^2 grid whatever they do, 22 us per iteration and solve, and a
// batch's spectra go through HBM three times per iteration.  Where the three
// strain components of a solve fit one CU's LDS, one workgroup keeps them there
// and iterates on its own until the stopping rule is met: C2R, Hooke's law and
// R2C along x, the transforms along y with the Green update between them, and
// the FP64 residual sum.  HBM (in fact L2) only sees the state and the force.
//
// Component c is stored as complex rows [y][kx] of pitch LP.  Both transforms run
// in place on it, a wave taking whole rows, then whole columns: the Stockham
// passes gather a butterfly's points into registers and scatter them when the
// wave has read its own.  A lane takes the same butterfly of all three
// components next to Hooke's law and to the Green update, which need them
// together.  Grids of more rows or columns than the waves hold at once are taken
// in rounds.
//
// LDS and FP64 arithmetic bound it, each busy for half the time (17.3 us per
// iteration of 64^2 in FP64; the LDS moves 19 sweeps of the three components and
// the twiddles, an iteration has 1430 FP64 instructions per wave).  One solve of
// 64^2 by 102 iterations takes 1772 us where its launches took 2250; 256 shifted
// solves take 2020 us for 5200.
#include "kernels_impl.hpp"
#include "launch.hpp"

namespace lsfft {
namespace {

// radix plans of the x transforms (half lengths): the pass next to Hooke's law
// holds three components, so the first forward radix is at most 4
template <int N> struct PlanX : Plan<N> {};
template <> struct PlanX<8> { static constexpr int np = 2, r0 = 4, r1 = 2, r2 = 1; };
template <> struct PlanX<24> { static constexpr int np = 3, r0 = 4, r1 = 2, r2 = 3; };
template <> struct PlanX<64> { static constexpr int np = 3, r0 = 4, r1 = 4, r2 = 4; };

constexpr int NT2 = 512;
constexpr int NC = 3;    // strain components
// Padding of a row of spectra: with four entries a wave's columns of the y passes
// of power-of-two lengths meet no bank twice.
constexpr int kPad2d = 4;
// Largest solve taken.  One CU's time grows with the points, the launches' hardly
// does: per iteration in FP64 7.1 against 19 us at 16^2, 17.6 against 21.6 at
// 64^2, 24.8 against 24.9 at 256 x 16, but 31 against 25.6 at 64 x 96 (FP32: 15.8
// against 25 at 64^2, 27 against 24 at 64 x 96).  Up to here it all fits LDS: 156
// KB for 256 rows of 16 points in FP64 and 256 phases.
constexpr int kPoints2d = 4096;

template <typename T> using V2 = T __attribute__((ext_vector_type(2)));

// Passes of a length-N transform of all components of the MP pencils that a wave
// owns.  `at` maps (component, pencil, index) to an LDS word.
//  JF: index-fastest butterflies (x), else pencil-fastest (y)
// A wave's LDS operations are in order, so its passes need no barrier, and one
// wave's LDS traffic overlaps another's arithmetic: with workgroup barriers
// between the passes (rows and columns dealt to all waves) the two added up, 20.0
// us per iteration of 64^2 in FP64 where this takes 17.3.
// The chain pass (the one that meets the pointwise stage: the inverse x
// transform's last and the forward one's first, the forward y transform's last
// and the inverse one's first) has one butterfly of every component per thread;
// the others deal all components' butterflies out evenly.
template <typename T, int N, int DIR, bool REV, template <int> class PL, bool JF, int MP, int TWS, bool CHFIRST>
struct Fft3 {
  using S = PlanSeq<PL, N, REV>;
  static constexpr int np = S::np;
  template <int P> static constexpr bool chain() { return CHFIRST ? P == 0 : P == np - 1; }
  template <int P> static constexpr int tot() { return MP * (N / S::r(P)); }
  // butterflies per thread
  template <int P> static constexpr int bpt() { return chain<P>() ? NC : (NC * tot<P>() + 63) / 64; }

  // butterfly q of this thread: component, pencil, index
  template <int P>
  __device__ static __forceinline__ bool where(int tid, int q, int npen, int& c, int& m, int& j) {
    constexpr int NB = N / S::r(P), TOT = tot<P>();
    int b;
    if constexpr (chain<P>()) {
      static_assert(TOT <= 64, "one chain butterfly per lane");
      c = q;
      b = tid;
    } else {
      if constexpr (TOT % 64 == 0) {   // a lane's butterflies: the same of each component
        c = q / (TOT / 64);
        b = tid + 64 * (q % (TOT / 64));
      } else {
        const int id = tid + q * 64;
        c = id / TOT;
        b = id - c * TOT;
      }
    }
    if constexpr (JF) {
      m = b / NB;
      j = b - m * NB;
    } else {
      m = b % MP;
      j = b / MP;
    }
    return (TOT % 64 == 0 || (c < NC && b < TOT)) && m < npen;
  }
  template <int P, typename A>
  __device__ static __forceinline__ void gather(T (&vr)[bpt<P>()][S::r(P)], T (&vi)[bpt<P>()][S::r(P)], const V2<T>* z,
                                                const A& at, int npen, int tid) {
#pragma unroll
    for (int q = 0; q < bpt<P>(); ++q) {
      int c, m, j;
      const bool ok = where<P>(tid, q, npen, c, m, j);
#pragma unroll
      for (int r = 0; r < S::r(P); ++r) {
        const int i = ok ? at(c, m, j + r * (N / S::r(P))) : 0;
        const V2<T> v = z[i];
        vr[q][r] = v.x;
        vi[q][r] = v.y;
      }
    }
  }
  // twiddles and butterflies of pass P
  template <int P>
  __device__ static __forceinline__ void compute(T (&vr)[bpt<P>()][S::r(P)], T (&vi)[bpt<P>()][S::r(P)], const V2<T>* tw,
                                                 int npen, int tid) {
    constexpr int RR = S::r(P), NS = S::ns(P);
#pragma unroll
    for (int q = 0; q < bpt<P>(); ++q) {
      if constexpr (NS > 1) {
        int c, m, j;
        where<P>(tid, q, npen, c, m, j);
        const int k = j % NS;
#pragma unroll
        for (int r = 1; r < RR; ++r) {
          const int t = r * k * (N / (NS * RR)) * TWS;
          const V2<T> w = tw[t];
          cmul(vr[q][r], vi[q][r], w.x, (DIR < 0) ? w.y : -w.y);
        }
      }
      bfly<T, RR, DIR>(vr[q], vi[q]);
    }
  }
  // outputs to their autosorted places (the last pass: j + r N / R)
  template <int P, typename A>
  __device__ static __forceinline__ void scatter(const T (&vr)[bpt<P>()][S::r(P)], const T (&vi)[bpt<P>()][S::r(P)],
                                                 V2<T>* z, const A& at, int npen, int tid) {
    constexpr int RR = S::r(P), NS = S::ns(P);
#pragma unroll
    for (int q = 0; q < bpt<P>(); ++q) {
      int c, m, j;
      if (where<P>(tid, q, npen, c, m, j)) {
        const int base = (j / NS) * NS * RR + (j % NS);
#pragma unroll
        for (int r = 0; r < RR; ++r) {
          const int i = at(c, m, base + r * NS);
          z[i] = V2<T>{vr[q][r], vi[q][r]};
        }
      }
    }
  }
  // inputs of the first pass in registers -> outputs of the last in registers
  template <typename A>
  __device__ static __forceinline__ void run(T (&ir)[bpt<0>()][S::r(0)], T (&ii)[bpt<0>()][S::r(0)],
                                             T (&o_r)[bpt<np - 1>()][S::r(np - 1)],
                                             T (&o_i)[bpt<np - 1>()][S::r(np - 1)], V2<T>* z, const A& at,
                                             const V2<T>* tw, int npen, int tid) {
    compute<0>(ir, ii, tw, npen, tid);
    if constexpr (np == 1) {
      static_assert(np > 1 || chain<0>(), "single-pass transforms chain");
#pragma unroll
      for (int q = 0; q < bpt<0>(); ++q)
#pragma unroll
        for (int r = 0; r < S::r(0); ++r) {
          o_r[q][r] = ir[q][r];
          o_i[q][r] = ii[q][r];
        }
    } else {
      wave_order();
      scatter<0>(ir, ii, z, at, npen, tid);
      wave_order();
      if constexpr (np == 3) {
        T mr[bpt<1>()][S::r(1)], mi[bpt<1>()][S::r(1)];
        gather<1>(mr, mi, z, at, npen, tid);
        compute<1>(mr, mi, tw, npen, tid);
        wave_order();
        scatter<1>(mr, mi, z, at, npen, tid);
        wave_order();
      }
      gather<np - 1>(o_r, o_i, z, at, npen, tid);
      compute<np - 1>(o_r, o_i, tw, npen, tid);
    }
  }
};

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// shared state of a solve
template <typename T> struct Lds {
  V2<T>* z;                // [NC][ny][LP]
  V2<T> *twx, *twy;
  T *lam, *mu;
  const uint8_t* ph;       // [ny][nx], shifted
  int LP, CS;              // row pitch, component stride
};

// strain spectra -> strain, Hooke's law, stress -> spectra, row chunk by row chunk
template <typename T, int NX>
__device__ __forceinline__ void x_phase(const Lds<T>& L, int ny) {
  constexpr int H = NX / 2;
  constexpr int RP = PlanX<H>::r0, MR = 64 / (H / RP);
  using FI = Fft3<T, H, +1, true, PlanX, true, MR, 2, false>;
  using FF = Fft3<T, H, -1, false, PlanX, true, MR, 2, true>;
  constexpr int P0 = FI::S::r(0), PL_ = FF::S::r(FF::np - 1);
  static_assert(FI::S::r(FI::np - 1) == RP && FF::S::r(0) == RP, "x transforms chain in registers");
  for (int y0 = MR * wave_id(); y0 < ny; y0 += MR * (NT2 / 64)) {
    const int nr = min(MR, ny - y0);
    // opaque: addresses are formed where they are used; kept across iterations
    // they fill the registers
    int tid = threadIdx.x & 63;
    asm volatile("" : "+v"(tid));
    auto at = [&](int c, int m, int n) { return c * L.CS + (y0 + m) * L.LP + n; };
    T vr[NC][RP], vi[NC][RP];
    {
      T ir[FI::template bpt<0>()][P0], ii[FI::template bpt<0>()][P0];
#pragma unroll
      for (int q = 0; q < FI::template bpt<0>(); ++q) {
        int c, m, j;
        const bool ok = FI::template where<0>(tid, q, nr, c, m, j);
#pragma unroll
        for (int r = 0; r < P0; ++r) {
          const int k = ok ? j + r * (H / P0) : 0;
          // the packed entry X[0] + i X[H] at k = 0
          const int a = ok ? at(c, m, k) : 0, b = ok ? at(c, m, k ? H - k : 0) : 0;
          const V2<T> va = L.z[a], vb = L.z[b], w = L.twx[k];
          T xr = va.x, xi = va.y, yr = vb.x, yi = -vb.y;
          if (r == 0 && k == 0) {
            yr = xi;
            yi = T(0);
            xi = T(0);
          }
          const T dr = xr - yr, di = xi - yi;
          const T cr = w.x, ci = -w.y;
          const T tr = cr * dr - ci * di, ti = cr * di + ci * dr;
          ir[q][r] = xr + yr - ti;
          ii[q][r] = xi + yi + tr;
        }
      }
      FI::run(ir, ii, vr, vi, L.z, at, L.twx, nr, tid);
    }
    {
      int c0_, m, j;
      if (FF::template where<0>(tid, 0, nr, c0_, m, j)) {
        const uint8_t* ph = L.ph + (y0 + m) * NX;
#pragma unroll
        for (int r = 0; r < RP; ++r) {
          const int n = j + r * (H / RP);
          const unsigned pp = *reinterpret_cast<const unsigned short*>(ph + 2 * n);
          const T l0 = L.lam[pp & 0xffu], m0 = L.mu[pp & 0xffu], l1 = L.lam[pp >> 8], m1 = L.mu[pp >> 8];
          const T t0 = l0 * (vr[0][r] + vr[1][r]), t1 = l1 * (vi[0][r] + vi[1][r]);
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            vr[c][r] = T(2) * m0 * vr[c][r] + (c < 2 ? t0 : T(0));
            vi[c][r] = T(2) * m1 * vi[c][r] + (c < 2 ? t1 : T(0));
          }
        }
      }
    }
    {
      T zr[FF::template bpt<FF::np - 1>()][PL_], zi[FF::template bpt<FF::np - 1>()][PL_];
      FF::run(vr, vi, zr, zi, L.z, at, L.twx, nr, tid);
      wave_order();
      FF::template scatter<FF::np - 1>(zr, zi, L.z, at, nr, tid);
    }
    wave_order();
    // unfold in place, the pair (k, H - k) by one lane; 0 goes with H / 2
    for (int e = tid; e < nr * (H / 2); e += 64) {
      const int m = e / (H / 2), k = e - m * (H / 2), kb = k ? H - k : H / 2;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int a = at(c, m, k), b = at(c, m, kb);
        const V2<T> va = L.z[a], vb = L.z[b];
        auto half = [&](V2<T> z, V2<T> w, V2<T> t) {
          const T er = T(0.5) * (z.x + w.x), ei = T(0.5) * (z.y - w.y);
          const T orr = T(0.5) * (z.y + w.y), oi = T(-0.5) * (z.x - w.x);
          return V2<T>{er + t.x * orr - t.y * oi, ei + t.x * oi + t.y * orr};
        };
        const V2<T> xa = half(va, vb, L.twx[k]);
        L.z[b] = half(vb, k ? va : vb, L.twx[kb]);
        L.z[a] = k ? xa : V2<T>{va.x + va.y, va.x - va.y};
      }
    }
    wave_order();
  }
  lds_barrier();
}

// stress spectra -> residual, update of the state, next strain spectra; returns
// this thread's share of the residual sum
template <typename T, int NY>
__device__ __forceinline__ double y_phase(const Lds<T>& L, const InstDesc& D, int cur) {
  constexpr int RP = PlanSeq<PlanG, NY, false>::last(), MC = 64 / (NY / RP);
  using FF = Fft3<T, NY, -1, false, PlanG, false, MC, 1, false>;
  using FI = Fft3<T, NY, +1, true, PlanG, false, MC, 1, true>;
  constexpr int P0 = FF::S::r(0), PE = FI::S::r(FI::np - 1);
  static_assert(FF::S::r(FF::np - 1) == RP && FI::S::r(0) == RP, "y transforms chain in registers");
  const int H = D.H;
  const long long Pc = D.Pc;
  const T inv_n = T(D.inv_nvox), mu0 = T(D.mu0);
  const T c0 = T((D.lam0 + D.mu0) / (D.lam0 + 2.0 * D.mu0));
  double part = 0.0;
  for (int k0 = MC * wave_id(); k0 < H; k0 += MC * (NT2 / 64)) {
    const int nc = min(MC, H - k0);
    int tid = threadIdx.x & 63;
    asm volatile("" : "+v"(tid));
    auto at = [&](int c, int m, int n) { return c * L.CS + n * L.LP + k0 + m; };
    int c_, m, j;
    const bool ok = FI::template where<0>(tid, 0, nc, c_, m, j);
    // force and state of this thread's points, in flight during the transform
    V2<T> fv[2][RP], uv[2][RP];
    if (ok) {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int r = 0; r < RP; ++r) {
          const unsigned g = (unsigned)((j + r * (NY / RP)) * H + k0 + m);
          fv[a][r] = gld<V2<T>>(cptr<T>(D.F, Pc, a), g);
          uv[a][r] = gld<V2<T>>(cptr<T>(D.U[cur], Pc, a), g);
        }
    }
    T sr[NC][RP], si[NC][RP];
    {
      T ir[FF::template bpt<0>()][P0], ii[FF::template bpt<0>()][P0];
      FF::template gather<0>(ir, ii, L.z, at, nc, tid);
      FF::run(ir, ii, sr, si, L.z, at, L.twy, nc, tid);
    }
    if (ok) {
      const T xi0 = T(wavenum(k0 + m, D.nx, D.kx));
      const double w = (k0 + m == 0) ? 1.0 : 2.0;
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        const int n = j + r * (NY / RP);
        const T xi[2] = {xi0, T(wavenum(n, NY, D.ky))};
        const T xi2 = xi[0] * xi[0] + xi[1] * xi[1];
        // r = i xi . sigma^ + f^
        T vr[2], vi[2];
        vr[0] = fv[0][r].x - (xi[0] * si[0][r] + xi[1] * si[2][r]);
        vi[0] = fv[0][r].y + (xi[0] * sr[0][r] + xi[1] * sr[2][r]);
        vr[1] = fv[1][r].x - (xi[0] * si[2][r] + xi[1] * si[1][r]);
        vi[1] = fv[1][r].y + (xi[0] * sr[2][r] + xi[1] * sr[1][r]);
#pragma unroll
        for (int a = 0; a < 2; ++a)
          part += w * (double(vr[a]) * double(vr[a]) + double(vi[a]) * double(vi[a]));
        apply_n0<T, 2>(xi, xi2, c0, mu0, vr, vi);
        const unsigned g = (unsigned)(n * H + k0 + m);
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          vr[a] += uv[a][r].x;
          vi[a] += uv[a][r].y;
          stc<T>(mptr<T>(D.U[cur ^ 1], Pc, a), g, vr[a], vi[a]);
        }
        // eps^_ab = (i / 2)(xi_a u^_b + xi_b u^_a) / |N|
        sr[0][r] = -(xi[0] * vi[0]) * inv_n;
        si[0][r] = (xi[0] * vr[0]) * inv_n;
        sr[1][r] = -(xi[1] * vi[1]) * inv_n;
        si[1][r] = (xi[1] * vr[1]) * inv_n;
        sr[2][r] = -(T(0.5) * (xi[0] * vi[1] + xi[1] * vi[0])) * inv_n;
        si[2][r] = (T(0.5) * (xi[0] * vr[1] + xi[1] * vr[0])) * inv_n;
      }
    }
    T er[FI::template bpt<FI::np - 1>()][PE], ei[FI::template bpt<FI::np - 1>()][PE];
    FI::run(sr, si, er, ei, L.z, at, L.twy, nc, tid);
    wave_order();
    FI::template scatter<FI::np - 1>(er, ei, L.z, at, nc, tid);
  }
  lds_barrier();
  return part;
}

#define LSFFT_LENS2D(X) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(256)

template <typename T>
__global__ __launch_bounds__(NT2) void k_solve2d(const InstDesc* __restrict__ descs, InstState* states,
                                                 const int* __restrict__ inst, const double* __restrict__ lame,
                                                 const T* __restrict__ tw, int steps) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double red[NT2 / 64];
  __shared__ InstState state;   // this solve's, written back when the launch ends
  const int tid = threadIdx.x;
  const InstDesc& D = descs[inst[blockIdx.x]];
  if (tid == 0) state = states[inst[blockIdx.x]];
  __syncthreads();
  if (state.status != ST_RUNNING) return;
  const int nx = D.nx, ny = D.ny, H = D.H;
  const long long Pc = D.Pc;
  Lds<T> L;
  L.LP = H + kPad2d;
  L.CS = ny * L.LP;
  L.z = reinterpret_cast<V2<T>*>(smem);
  L.twx = L.z + NC * L.CS;
  L.twy = L.twx + nx;
  L.lam = reinterpret_cast<T*>(L.twy + ny);
  L.mu = L.lam + D.nphase;
  uint8_t* ph = reinterpret_cast<uint8_t*>(L.mu + D.nphase);
  L.ph = ph;
  auto table = [&](int len, V2<T>* t) {
    int off = 0;
    for (int k = 0; k < kNumLens; ++k) {
      if (len_at(k) == len) break;
      off += len_at(k);
    }
    for (int k = tid; k < len; k += NT2) t[k] = reinterpret_cast<const V2<T>*>(tw)[off + k];
  };
  table(nx, L.twx);
  table(ny, L.twy);
  for (int p = tid; p < D.nphase; p += NT2) {
    L.lam[p] = T(lame[2 * (D.lame_off + p)]);
    L.mu[p] = T(lame[2 * (D.lame_off + p) + 1]);
  }
  for (int e = tid; e < nx * ny; e += NT2) {
    const int y = e / nx, x = e - y * nx;
    ph[e] = D.phase[(long long)wrap(y - D.sy, ny) * nx + wrap(x - D.sx, nx)];
  }
  for (int e = tid; e < ny * H; e += NT2) {
    const int y = e / H, k = e - y * H;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const typename C2<T>::type v = ldc<T>(cptr<T>(D.S, Pc, c), e);
      L.z[c * L.CS + y * L.LP + k] = V2<T>{v.x, v.y};
    }
  }
  __syncthreads();
  for (int step = 0; step < steps; ++step) {
    switch (nx) {
#define X(N) case N: x_phase<T, N>(L, ny); break;
      LSFFT_LENS2D(X)
#undef X
    }
    double part = 0.0;
    const int cur = state.iter & 1;
    switch (ny) {
#define X(N) case N: part = y_phase<T, N>(L, D, cur); break;
      LSFFT_LENS2D(X)
#undef X
    }
    const double sum = block_sum<NT2>(part, red);
    if (tid == 0) judge(D, state, sqrt(sum / state.fnorm2));
    __syncthreads();   // also: this iteration's state is in memory for the next one's loads
    if (state.status != ST_RUNNING) break;
  }
  if (tid == 0) states[inst[blockIdx.x]] = state;
  if (state.status != ST_RUNNING) return;
  // out of steps: leave the strain spectra for the next launch
  for (int e = tid; e < ny * H; e += NT2) {
    const int y = e / H, k = e - y * H;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const V2<T> v = L.z[c * L.CS + y * L.LP + k];
      stc<T>(mptr<T>(D.S, Pc, c), e, v.x, v.y);
    }
  }
}

}  // namespace

size_t solve2d_lds(bool f64, int nx, int ny, int nphase) {
  auto listed = [](int n) {
    switch (n) {
#define X(N) case N:
      LSFFT_LENS2D(X)
#undef X
      return true;
      default: return false;
    }
  };
  if (!listed(nx) || !listed(ny)) return 0;
  if (nx * ny > kPoints2d || nphase > 256) return 0;
  const size_t ts = f64 ? 8 : 4;
  return (ts * ((size_t)2 * NC * ny * (nx / 2 + kPad2d) + 2 * (nx + ny) + 2 * nphase) + (size_t)nx * ny + 15) / 16 * 16;
}

hipError_t launch_solve2d(bool f64, const LaunchArgs& a, const int* inst, int count, int steps) {
  if (count <= 0) return hipSuccess;
  if (a.lds > (size_t)kMaxDynamicLds) return hipErrorInvalidValue;
  const void* k = f64 ? reinterpret_cast<const void*>(k_solve2d<double>) : reinterpret_cast<const void*>(k_solve2d<float>);
  const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxDynamicLds);
  if (e != hipSuccess) return e;
  if (f64)
    hipLaunchKernelGGL(k_solve2d<double>, dim3((unsigned)count), NT2, a.lds, a.stream, a.desc, a.state, inst, a.lame,
                       static_cast<const double*>(a.tw), steps);
  else
    hipLaunchKernelGGL(k_solve2d<float>, dim3((unsigned)count), NT2, a.lds, a.stream, a.desc, a.state, inst, a.lame,
                       static_cast<const float*>(a.tw), steps);
  return hipGetLastError();
}

}  // namespace lsfft
