// The y and x transforms of an iteration in one pass over z planes: inverse y,
// C2R along x, Hooke's law, R2C along x and forward y of one plane of three strain
// components (the normal ones, which the trace couples, or the shears) by one
// workgroup.
//
// As three launches (k_ypass, k_xpass, k_ypass) the spectra go through memory six
// times, 36 half-spectrum streams of an iteration's 57; here once in and once out,
// 12.  A component's plane sits in LDS while it is transformed, one after another;
// the real strains of the three wait in registers for Hooke's law.  Every wave owns
// whole columns, then whole rows: its passes need no workgroup barrier, and its LDS
// traffic overlaps other waves' arithmetic.  The next component's plane is loaded
// into registers meanwhile.
//
// What bounds it is arithmetic and LDS, busy for 52 to 70 and 52 to 63 % of the time
// (without packed FP32 a wave's FP32 instruction takes four cycles; an LDS sweep of
// the plane per pass and direction, 23 in all).  Measured for FP32, per launch: 47.5
// us at 128^3 where the three passes took 76.7 (26.8 + 31.9 + 18.0), 62 us against
// 116 for sixteen solves of 64^3, 67.5 against 88 for as many of 96^3.  Half of the
// instructions were address arithmetic at first (49.8 us at 128^3, 18.3 million
// wave-instructions against 13.5): hence the constants apart wherever no carry
// occurs, and lanes whose range the compiler knows.
//
// The roundings are those of the three passes, instruction for instruction (the
// radix plans, the order of every sum, which product of a complex multiplication is
// fused), so that both ways give the same bits.
#include <algorithm>

#include "kernels_impl.hpp"
#include "launch.hpp"

namespace lsfft {
namespace {

template <typename T> using V2 = T __attribute__((ext_vector_type(2)));

// a b, rounded as in the other passes
__device__ __forceinline__ void cmul_fma(float& ar, float& ai, float br, float bi) {
  const float t = __builtin_fmaf(ar, br, -(ai * bi));
  ai = __builtin_fmaf(ai, br, ar * bi);
  ar = t;
}

// Passes of a length-N transform of the MP pencils that a wave owns.
//  JF: index-fastest butterflies (x), else pencil-fastest (y)
//  entry n of a pencil: word base + n P_ + (n / 8) Q_; with the step after every 8
//  the strided scatters of the first passes spread over the banks
template <typename T, int N, int DIR, bool REV, template <int> class PL, bool JF, int MP, int P_, int Q_, int TWS>
struct WaveFft {
  using S = PlanSeq<PL, N, REV>;
  static constexpr int np = S::np;
  template <int P> static constexpr int tot() { return MP * (N / S::r(P)); }
  template <int P> static constexpr int bpt() { return (tot<P>() + 63) / 64; }
  static constexpr int word(int n) { return n * P_ + (n >> 3) * Q_; }
  // butterfly q of this lane
  template <int P> __device__ static __forceinline__ bool where(int lane, int q, int& m, int& j) {
    constexpr int NB = N / S::r(P);
    const int b = lane + 64 * q;
    if constexpr (JF) {
      m = b / NB;
      j = b - m * NB;
    } else {
      m = b % MP;
      j = b / MP;
    }
    if constexpr (tot<P>() % 64 == 0) return true;
    return b < tot<P>();
  }
  template <int P, typename B>
  __device__ static __forceinline__ void gather(T (&vr)[bpt<P>()][S::r(P)], T (&vi)[bpt<P>()][S::r(P)], const V2<T>* z,
                                                const B& base, int lane) {
    constexpr int RR = S::r(P), NB = N / RR;
#pragma unroll
    for (int q = 0; q < bpt<P>(); ++q) {
      int m, j;
      const bool ok = where<P>(lane, q, m, j);
      const V2<T>* a = z + (ok ? base(m) + (NB % 8 == 0 ? word(j) : 0) : 0);
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        const V2<T> v = a[NB % 8 == 0 ? word(r * NB) : (ok ? word(j + r * NB) : 0)];
        vr[q][r] = v.x;
        vi[q][r] = v.y;
      }
    }
  }
  template <int P>
  __device__ static __forceinline__ void compute(T (&vr)[bpt<P>()][S::r(P)], T (&vi)[bpt<P>()][S::r(P)],
                                                 const V2<T>* tw, int lane) {
    constexpr int RR = S::r(P), NS = S::ns(P);
#pragma unroll
    for (int q = 0; q < bpt<P>(); ++q) {
      if constexpr (NS > 1) {
        int m, j;
        where<P>(lane, q, m, j);
        const int t = (j % NS) * (N / (NS * RR)) * TWS;
#pragma unroll
        for (int r = 1; r < RR; ++r) {
          const V2<T> w = tw[r * t];
          cmul_fma(vr[q][r], vi[q][r], w.x, (DIR < 0) ? w.y : -w.y);
        }
      }
      bfly<T, RR, DIR>(vr[q], vi[q]);
    }
  }
  template <int P, typename B>
  __device__ static __forceinline__ void scatter(const T (&vr)[bpt<P>()][S::r(P)], const T (&vi)[bpt<P>()][S::r(P)],
                                                 V2<T>* z, const B& base, int lane) {
    constexpr int RR = S::r(P), NS = S::ns(P);
    // no carry into n / 8 within a butterfly: its words are constants apart
    constexpr bool flat = NS % 8 == 0 || (8 % NS == 0 && ((NS * RR) % 8 == 0 || NS * RR == 4 || NS * RR == 2));
#pragma unroll
    for (int q = 0; q < bpt<P>(); ++q) {
      int m, j;
      if (where<P>(lane, q, m, j)) {
        const int n0 = (j / NS) * NS * RR + (j % NS);
        V2<T>* a = z + base(m) + (flat ? word(n0) : 0);
#pragma unroll
        for (int r = 0; r < RR; ++r) a[flat ? word(r * NS) : word(n0 + r * NS)] = V2<T>{vr[q][r], vi[q][r]};
      }
    }
  }
  // passes after the first butterflies' inputs are in registers, up to the last
  // pass's outputs in registers
  template <typename B>
  __device__ static __forceinline__ void run(T (&ir)[bpt<0>()][S::r(0)], T (&ii)[bpt<0>()][S::r(0)],
                                             T (&o_r)[bpt<np - 1>()][S::r(np - 1)],
                                             T (&o_i)[bpt<np - 1>()][S::r(np - 1)], V2<T>* z, const B& base,
                                             const V2<T>* tw, int lane) {
    static_assert(np == 2 || np == 3, "two or three passes");
    compute<0>(ir, ii, tw, lane);
    wave_order();
    scatter<0>(ir, ii, z, base, lane);
    wave_order();
    if constexpr (np == 3) {
      T mr[bpt<1>()][S::r(1)], mi[bpt<1>()][S::r(1)];
      gather<1>(mr, mi, z, base, lane);
      compute<1>(mr, mi, tw, lane);
      wave_order();
      scatter<1>(mr, mi, z, base, lane);
      wave_order();
    }
    gather<np - 1>(o_r, o_i, z, base, lane);
    compute<np - 1>(o_r, o_i, tw, lane);
  }
  // in place, LDS to LDS
  template <typename B>
  __device__ static __forceinline__ void inplace(V2<T>* z, const B& base, const V2<T>* tw, int lane) {
    T ir[bpt<0>()][S::r(0)], ii[bpt<0>()][S::r(0)], o_r[bpt<np - 1>()][S::r(np - 1)], o_i[bpt<np - 1>()][S::r(np - 1)];
    gather<0>(ir, ii, z, base, lane);
    run(ir, ii, o_r, o_i, z, base, tw, lane);
    wave_order();
    scatter<np - 1>(o_r, o_i, z, base, lane);
  }
};

// Waves of a plane: a divisor w of the columns and of the rows, for which a lane
// holds 4 to 8 complex points and the butterflies of all passes leave
// the fewest lane slots; with as many, the more waves.
template <template <int> class PL, int N, int MP> constexpr int plan_slots() {
  using S = PlanSeq<PL, N, false>;
  int s = 0;
  for (int p = 0; p < S::np; ++p) s += (MP * (N / S::r(p)) + 63) / 64 * S::r(p);
  return s;
}
template <int NX, int NY, int W> constexpr int waves_cost() {
  constexpr int H = NX / 2;
  if constexpr (H % W != 0 || NY % W != 0) {
    return 1 << 30;
  } else {
    if (H * NY > 64 * W * 8 || H * NY < 64 * W * 4) return 1 << 30;
    return (plan_slots<Plan, H, NY / W>() + plan_slots<Plan, NY, H / W>()) * W;
  }
}
template <int NX, int NY> constexpr int plane_waves() {
  const int w[10] = {16, 12, 10, 8, 6, 5, 4, 3, 2, 1};
  const int c[10] = {waves_cost<NX, NY, 16>(), waves_cost<NX, NY, 12>(), waves_cost<NX, NY, 10>(),
                     waves_cost<NX, NY, 8>(),  waves_cost<NX, NY, 6>(),  waves_cost<NX, NY, 5>(),
                     waves_cost<NX, NY, 4>(),  waves_cost<NX, NY, 3>(),  waves_cost<NX, NY, 2>(),
                     waves_cost<NX, NY, 1>()};
  int best = 0;
  for (int i = 1; i < 10; ++i)
    if (c[i] < c[best]) best = i;
  return c[best] < (1 << 30) ? w[best] : 0;
}

// Plane geometry: entry (y, kx) at word y P + (y / 8) Q + kx + kx / 8.  The row
// pitch and the step after 8 rows are odd multiples of a wave's columns (rounded up
// to a power of two), so that the columns of several rows fill the banks.
template <typename T, int NX, int NY> struct PlaneCfg {
  static constexpr int H = NX / 2;
  static constexpr int W = plane_waves<NX, NY>();
  static_assert(W > 0, "a wave count for these lengths");
  static constexpr int NT = 64 * W, CW = H / W, RW = NY / W;
  static constexpr int EU = (NX % 3 == 0 || NY % 3 == 0) && W < 16 ? 3 : 4;   // waves per SIMD
  // ... where there are more planes than CUs.  At three waves per SIMD a second
  // workgroup of six waves does not get in beside the first: 48 x 96, six solves of
  // 48 planes, 139 us per iteration (the three passes 123), with four waves 123, of 96
  // planes 217 (204) and 190.  For one solve of 48 planes, 57 against 61 us (65), the
  // registers of three waves.
  static constexpr int EUB = W > 4 && W % 4 != 0 ? 4 : EU;
  static constexpr int p2(int n) { int p = 1; while (p < n) p *= 2; return p; }
  static constexpr int Q = p2(CW) < 16 ? p2(CW) : 16;
  static constexpr int HP = H + H / 8;
  static constexpr int P = (HP - Q + 2 * Q - 1) / (2 * Q) * (2 * Q) + Q;
  static_assert(P >= HP && P % (2 * Q) == Q, "row pitch");
  static constexpr int WORDS = NY * P + NY / 8 * Q;
  // A plane whose workgroup has a CU to itself takes two buffers in turn, which saves
  // the barrier between one component's last reads and the next one's first writes.
  static constexpr int NBUF = W > 8 ? 2 : 1;
  static constexpr size_t LDS = sizeof(T) * ((size_t)2 * (NBUF * WORDS + NX + NY) + 2 * 256);
  static_assert(LDS <= 158 * 1024, "LDS");
};

// reduce_solve with its order of summation for NTH threads, by NT threads
template <int NTH, int NT>
__device__ inline void reduce_solve_by(const InstDesc& D, InstState& St, double* red) {
  if (St.status != ST_RUNNING) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int vw = wave; vw < NTH / 64; vw += NT / 64) {
    double a = 0.0;
    for (int k = vw * 64 + lane; k < D.items_g; k += NTH) a += D.partial[2 * k];
    for (int off = 32; off > 0; off >>= 1) a += __shfl_down(a, off, 64);
    if (lane == 0) red[vw] = a;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < NTH / 64; ++w) s += red[w];
    InstState loc = St;
    finalize(D, loc, M_ITER, s, 0.0);
    St = loc;
  }
}

// X[k] from Z[k], Z[H - k] and the twiddle, rounded as the x pass rounds it
__device__ __forceinline__ V2<float> unfold(V2<float> z, V2<float> w, V2<float> t) {
#pragma clang fp contract(off)
  const float orr = 0.5f * (z.y + w.y), oi = -(0.5f * (z.x - w.x));
  V2<float> x;
  x.x = __builtin_fmaf(-t.y, oi, __builtin_fmaf(0.5f, z.x + w.x, t.x * orr));
  x.y = __builtin_fmaf(t.y, orr, __builtin_fmaf(0.5f, z.y - w.y, t.x * oi));
  return x;
}

// A copy that the compiler does not connect with the original: addresses formed
// from it are not kept from one component, or from one transform, to the next,
// where those of all sweeps together fill the registers.
template <int LIMIT> __device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  __builtin_assume(v >= 0 && v < LIMIT);
  return v;
}

template <typename T, int NX, int NY>
__device__ __forceinline__ void plane_item(const InstDesc& D, int local, const T* lam, const T* mu, V2<T>* zb,
                                           const V2<T>* twx, const V2<T>* twy) {
  using C = PlaneCfg<T, NX, NY>;
  constexpr int H = C::H, NT = C::NT;
  using YI = WaveFft<T, NY, +1, true, Plan, false, C::CW, C::P, C::Q, 1>;
  using YF = WaveFft<T, NY, -1, false, Plan, false, C::CW, C::P, C::Q, 1>;
  using XI = WaveFft<T, H, +1, true, Plan, true, C::RW, 1, 1, 2>;
  using XF = WaveFft<T, H, -1, false, Plan, true, C::RW, 1, 1, 2>;
  constexpr int RP = XF::S::r(0), BP = XF::template bpt<0>();
  static_assert(XI::S::r(XI::np - 1) == RP && XI::template bpt<XI::np - 1>() == BP, "x transforms chain in registers");
  constexpr int E = 16 / (int)sizeof(V2<T>);          // entries of a 16-byte piece
  constexpr int PR = H / E, NP = NY * PR, LB = (NP + NT - 1) / NT;   // pieces per row, per plane, per thread
  typedef T Piece __attribute__((ext_vector_type(2 * E)));
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = local >= D.nz, zz = local - (g ? D.nz : 0);
  // (a + b) / 8 split into a wave's part and a lane's wherever no carry can occur
  auto col = [&](int m) {
    const int k0 = wave * C::CW;
    if constexpr (C::CW % 8 == 0 || 8 % C::CW == 0) return k0 + (k0 >> 3) + m + (m >> 3);
    else return k0 + m + ((k0 + m) >> 3);
  };
  auto row = [&](int m) {
    const int y0 = wave * C::RW;
    if constexpr (C::RW % 8 == 0) return y0 * C::P + (y0 >> 3) * C::Q + (m * C::P + (m >> 3) * C::Q);
    else return (y0 + m) * C::P + ((y0 + m) >> 3) * C::Q;
  };
  // pieces of this thread: entries in memory and words in LDS
  const int sy = D.blk ? D.bls : H;   // entries from one y line to the next
  auto piece = [&](int t, int i, unsigned& a, int& w) {
    constexpr int YS = NT / PR;
    constexpr bool whole = NT % PR == 0 && YS % 8 == 0;
    const int e = whole ? t : t + i * NT, y = e / PR, k = (e - y * PR) * E;
    a = D.blk ? (unsigned)(((k >> 3) * NY + y) * sy + 8 * zz + (k & 7)) : (unsigned)((zz * NY + y) * sy + k);
    w = y * C::P + (y >> 3) * C::Q + k + (k >> 3);
    if constexpr (whole) {
      a += (unsigned)(i * YS * sy);
      w += i * (YS * C::P + YS / 8 * C::Q);
    }
    return NP % NT == 0 || t + i * NT < NP;
  };
  void* const SS = D.blk ? D.S2 : D.S;
  Piece pre[LB];
  auto fetch = [&](int c) {
    const char* s = cptr<T>(SS, D.Pc, 3 * g + c);
    const int t = fresh<NT>(tid);
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      unsigned a;
      int w;
      if (piece(t, i, a, w)) pre[i] = *reinterpret_cast<const LSFFT_GLOBAL Piece*>((const LSFFT_GLOBAL char*)s + (size_t)a * sizeof(V2<T>));
    }
  };
  fetch(0);
  // phase ids of this lane's points, two per entry
  unsigned ids[BP][RP];
  {
    const LSFFT_GLOBAL uint8_t* ph = (const LSFFT_GLOBAL uint8_t*)D.phase + (long long)wrap(zz - D.sz, D.nz) * (NX * NY);
#pragma unroll
    for (int q = 0; q < BP; ++q) {
      int m, j;
      const bool ok = XF::template where<0>(tid & 63, q, m, j);
      const LSFFT_GLOBAL uint8_t* pr = ph + wrap((ok ? wave * C::RW + m : 0) - D.sy, NY) * NX;
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        const int n = ok ? j + r * (H / RP) : 0;
        ids[q][r] = pr[wrap(2 * n - D.sx, NX)] | ((unsigned)pr[wrap(2 * n + 1 - D.sx, NX)] << 8);
      }
    }
  }
  T hr[3][BP][RP], hi[3][BP][RP];
#pragma unroll 1
  for (int c = 0; c < 3; ++c) {
    V2<T>* z = zb + (C::NBUF == 2 && c == 1 ? C::WORDS : 0);
    const int t = fresh<NT>(tid);
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      unsigned a;
      int w;
      if (piece(t, i, a, w)) {
        if constexpr (E == 2) {
          z[w] = V2<T>{pre[i][0], pre[i][1]};
          z[w + 1] = V2<T>{pre[i][2], pre[i][3]};
        } else {
          z[w] = V2<T>{pre[i][0], pre[i][1]};
        }
      }
    }
    lds_barrier();
    if (c < 2) fetch(c + 1);
    YI::inplace(z, col, twy, fresh<64>(tid & 63));
    lds_barrier();
    const int lane = fresh<64>(tid & 63);
    T vr[BP][RP], vi[BP][RP];
    {
      constexpr int P0 = XI::S::r(0), B0 = XI::template bpt<0>();
      T ir[B0][P0], ii[B0][P0];
#pragma unroll
      for (int q = 0; q < B0; ++q) {
        int m, j;
        const bool ok = XI::template where<0>(lane, q, m, j);
        const V2<T>* zr = z + (ok ? row(m) : 0);
#pragma unroll
        for (int r = 0; r < P0; ++r) {
          // the packed entry X[0] + i X[H] at k = 0, whose partner is not used
          constexpr int NB = H / P0;
          const int k = (ok ? j : 0) + r * NB;
          const int wa = NB % 8 == 0 ? XI::word(ok ? j : 0) + XI::word(r * NB) : XI::word(k);
          const int wb = NB % 8 == 0 ? XI::word(ok ? -j : 0) + XI::word(H - r * NB) : XI::word(k ? H - k : 0);
          const V2<T> va = zr[wa], vb = zr[wb], w = twx[k];
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
      XI::run(ir, ii, vr, vi, z, row, twx, lane);
    }
    // a uniform branch each: the code above exists once
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (c == d)
#pragma unroll
        for (int q = 0; q < BP; ++q)
#pragma unroll
          for (int r = 0; r < RP; ++r) {
            hr[d][q][r] = vr[q][r];
            hi[d][q][r] = vi[q][r];
          }
    if (C::NBUF == 1) lds_barrier();
  }
#pragma unroll
  for (int q = 0; q < BP; ++q)
#pragma unroll
    for (int r = 0; r < RP; ++r) {
      const unsigned pp = ids[q][r];
      const T l0 = lam[pp & 0xffu], m0 = mu[pp & 0xffu], l1 = lam[pp >> 8], m1 = mu[pp >> 8];
      const T t0 = g ? T(0) : l0 * (hr[0][q][r] + hr[1][q][r] + hr[2][q][r]);
      const T t1 = g ? T(0) : l1 * (hi[0][q][r] + hi[1][q][r] + hi[2][q][r]);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        hr[d][q][r] = __builtin_fmaf(T(2) * m0, hr[d][q][r], t0);
        hi[d][q][r] = __builtin_fmaf(T(2) * m1, hi[d][q][r], t1);
      }
    }
#pragma unroll 1
  for (int c = 0; c < 3; ++c) {
    V2<T>* z = zb + (C::NBUF == 2 && c != 1 ? C::WORDS : 0);
    const int lane = fresh<64>(tid & 63);
    T vr[BP][RP], vi[BP][RP];
#pragma unroll
    for (int q = 0; q < BP; ++q)
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        vr[q][r] = c == 0 ? hr[0][q][r] : c == 1 ? hr[1][q][r] : hr[2][q][r];
        vi[q][r] = c == 0 ? hi[0][q][r] : c == 1 ? hi[1][q][r] : hi[2][q][r];
      }
    {
      constexpr int PL = XF::S::r(XF::np - 1), BL = XF::template bpt<XF::np - 1>();
      T zr[BL][PL], zi[BL][PL];
      XF::run(vr, vi, zr, zi, z, row, twx, lane);
      wave_order();
      XF::template scatter<XF::np - 1>(zr, zi, z, row, lane);
    }
    wave_order();
    // unfold in place, the pair (k, H - k) by one lane; 0 goes with H / 2
    constexpr int UN = C::RW * (H / 2);
    constexpr bool same = 64 % (H / 2) == 0;   // a lane's pairs: the same in rows 128 / H apart
#pragma unroll
    for (int q = 0; q < (UN + 63) / 64; ++q) {
      const int e = same ? lane : lane + 64 * q, m = e / (H / 2) + (same ? q * (128 / H) : 0);
      const int k = e % (H / 2), kb = k ? H - k : H / 2;
      if (UN % 64 == 0 || lane + 64 * q < UN) {
        V2<T>* pa = z + row(m) + XF::word(k);
        V2<T>* pb = z + row(m) + XF::word(kb);
        const V2<T> va = *pa, vb = *pb;
        const V2<T> xa = unfold(va, vb, twx[k]);
        *pb = unfold(vb, k ? va : vb, twx[kb]);
        *pa = k ? xa : V2<T>{va.x + va.y, va.x - va.y};
      }
    }
    lds_barrier();
    YF::inplace(z, col, twy, fresh<64>(tid & 63));
    lds_barrier();
    const int t = fresh<NT>(tid);
    char* d = mptr<T>(SS, D.Pc, 3 * g + c);
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      unsigned a;
      int w;
      if (piece(t, i, a, w)) {
        Piece v;
        const V2<T> v0 = z[w];
        v[0] = v0.x;
        v[1] = v0.y;
        if constexpr (E == 2) {
          const V2<T> v1 = z[w + 1];
          v[2] = v1.x;
          v[3] = v1.y;
        }
        *reinterpret_cast<LSFFT_GLOBAL Piece*>((LSFFT_GLOBAL char*)d + (size_t)a * sizeof(V2<T>)) = v;
      }
    }
    if (C::NBUF == 1) lds_barrier();
  }
}

template <typename T, int NX, int NY, int EU>
__global__ __launch_bounds__((PlaneCfg<T, NX, NY>::NT)) __attribute__((amdgpu_waves_per_eu(EU))) void k_plane(
    const InstDesc* __restrict__ descs, InstState* states, const WorkItem* __restrict__ items,
    const int* __restrict__ nitems, const double* __restrict__ lame, const T* __restrict__ tw,
    const int* __restrict__ red_inst, const int* __restrict__ red_n) {
  using C = PlaneCfg<T, NX, NY>;
  constexpr int NT = C::NT;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double red[Cfg<T>::NTH / 64];
  __shared__ int s_run;
  V2<T>* z = reinterpret_cast<V2<T>*>(smem);
  V2<T>* twx = z + C::NBUF * C::WORDS;
  V2<T>* twy = twx + NX;
  T* lam = reinterpret_cast<T*>(twy + NY);
  if (red_n) {
    const int nr = *red_n;
    for (int r = blockIdx.x; r < nr; r += gridDim.x) {
      const int i = red_inst[r];
      reduce_solve_by<Cfg<T>::NTH, NT>(descs[i], states[i], red);
      __syncthreads();
    }
  }
  const int n_items = *nitems;
  if ((int)xcd_slot(blockIdx.x, gridDim.x) >= n_items) return;
  for (int k = threadIdx.x; k < NX; k += NT) twx[k] = reinterpret_cast<const V2<T>*>(tw)[tw_offset(NX) + k];
  for (int k = threadIdx.x; k < NY; k += NT) twy[k] = reinterpret_cast<const V2<T>*>(tw)[tw_offset(NY) + k];
  for (int w = xcd_slot(blockIdx.x, gridDim.x); w < n_items; w += gridDim.x) {
    const WorkItem it = items[w];
    const InstDesc& D = descs[it.inst];
    // one decision per workgroup: another one's prologue may change the status
    if (threadIdx.x == 0) s_run = (states[it.inst].status == ST_RUNNING);
    __syncthreads();
    const bool go = s_run != 0;
    __syncthreads();
    if (!go) continue;
    T* mu = lam + 256;   // a phase id is a byte
    for (int p = threadIdx.x; p < min(D.nphase, 256); p += NT) {
      lam[p] = T(lame[2 * (D.lame_off + p)]);
      mu[p] = T(lame[2 * (D.lame_off + p) + 1]);
    }
    plane_item<T, NX, NY>(D, it.local, lam, mu, z, twx, twy);
  }
}

#define LSFFT_PLANE_Y(X, T, NX) X(T, NX, 32) X(T, NX, 48) X(T, NX, 64) X(T, NX, 96) X(T, NX, 128)
#define LSFFT_PLANES(X, T) \
  LSFFT_PLANE_Y(X, T, 32) LSFFT_PLANE_Y(X, T, 48) LSFFT_PLANE_Y(X, T, 64) LSFFT_PLANE_Y(X, T, 96) LSFFT_PLANE_Y(X, T, 128)

constexpr int kCus = 256;
template <typename T, int NX, int NY, int EU> hipError_t launch_eu(const LaunchArgs& a) {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_plane<T, NX, NY, EU>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)a.lds);
  if (e != hipSuccess) return e;
  // as many workgroups as fit the chip at once: the launch is captured for the
  // batch's first iteration, and of the later ones' fewer solves the surplus
  // workgroups would each wait for a CU only to find nothing to do
  using C = PlaneCfg<T, NX, NY>;
  constexpr int kPerCu = 4 * EU / C::W < (int)(160 * 1024 / (C::LDS + 1024)) ? 4 * EU / C::W : (int)(160 * 1024 / (C::LDS + 1024));
  static_assert(kPerCu >= 1, "fits a CU");
  const dim3 grid(std::min<unsigned>(a.grid.x, kCus * kPerCu));
  LSFFT_LAUNCH((k_plane<T, NX, NY, EU>), grid, C::NT, a.lds, a.stream, a.desc, a.state, a.items,
               a.count, a.lame, static_cast<const T*>(a.tw), a.red_inst, a.red_n);
  return hipGetLastError();
}
template <typename T, int NX, int NY> hipError_t launch_one(const LaunchArgs& a) {
  using C = PlaneCfg<T, NX, NY>;
  if (C::EUB != C::EU && a.grid.x > kCus) return launch_eu<T, NX, NY, C::EUB>(a);
  return launch_eu<T, NX, NY, C::EU>(a);
}

}  // namespace

// Grids that take this path.  Planes of 128 x 96 points and more fill a CU each, and
// need about as many planes as pay for the 256 CUs: per iteration of one solve 85
// against 109 us for 96 planes of 128^2, 81 against 83.5 for 96 x 128, but 67.8
// against 66.4 and 72.5 against 61.7 us for 48.  Below, a launch of few planes takes
// as long as one plane: 46.8 against 44.1 us for 4 planes of 96^2, 49.5 against 49.4
// for 16, 57.6 against 63.1 for 48; 30.2 against 37.6 for 4 of 64^2.  In FP64 the
// three components' strains do not fit the registers: 41.4 us against 39.3 for 48
// planes of 96 x 64.
size_t plane_lds(bool f64, int nx, int ny, int nz) {
  if (f64 || !(nx * ny <= 4096 || (nx * ny <= 9216 && nz >= 16) || nz >= 96)) return 0;
#define X(T, NX, NY) \
  if (nx == NX && ny == NY) return PlaneCfg<T, NX, NY>::LDS;
  LSFFT_PLANES(X, float)
#undef X
  return 0;
}

hipError_t launch_plane(const LaunchArgs& a, int nx, int ny) {
#define X(T, NX, NY) \
  if (nx == NX && ny == NY) return launch_one<T, NX, NY>(a);
  LSFFT_PLANES(X, float)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace lsfft
