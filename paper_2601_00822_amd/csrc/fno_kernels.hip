// Kernels of the learned surrogate (Eq. 6.10 layers, Fourier-neural-operator
// family): pointwise layers and their gradients on bf16 MFMA
// (v_mfma_f32_32x32x16_bf16, fp32 accumulation), per-mode complex products
// on the same instruction, truncated transforms, loss and Adam in fp32.
//
// MFMA 32x32x16 operand layout used throughout (one wave, lane l):
//   A (32 x 16, row-major operand): row l % 32, columns 8 (l / 32) .. +7
//   B (16 x 32):                    column l % 32, rows 8 (l / 32) .. +7
//   C (32 x 32, 16 floats per lane): element e sits at
//       row 8 (e / 4) + 4 (l / 32) + e % 4, column l % 32.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fft_core.hpp"
#include "fno_launch.hpp"

namespace lsfft_fno {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NTB = 256;   // threads of the elementwise and transform kernels

__device__ __forceinline__ float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752440f)); }
__device__ __forceinline__ float gelu_grad(float x) {
  return 0.5f * (1.0f + erff(x * 0.70710678118654752440f)) + x * 0.39894228040143267794f * expf(-0.5f * x * x);
}

// both at once, sharing the error function
__device__ __forceinline__ void gelu_both(float x, float& z, float& g) {
  const float e = erff(x * 0.70710678118654752440f);
  z = 0.5f * x * (1.0f + e);
  g = 0.5f * (1.0f + e) + x * 0.39894228040143267794f * expf(-0.5f * x * x);
}

using lsfft::wave_order;

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 neg8(bf16x8 a) {
  bf16x8 r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r[j] = -a[j];
  return r;
}

template <typename K>
static hipError_t allow_lds(K kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             lsfft::kMaxDynamicLds);
}

// ---------------------------------------------------------------------------
// pointwise layer
// ---------------------------------------------------------------------------
// One wave per block of 32 NT voxels of one sample, computed as NT
// interleaved 32-column MFMA tiles: tile k holds voxels v0 + NT c + k
// (c = lane % 32), so every lane moves NT consecutive voxels, one per tile,
// in one vector access, and each half-wave reads or writes 128 NT
// contiguous bytes of one channel.  The B operand (input channels) is
// converted to bf16 once per block; the kWidth output channels (lift and hidden
// layers) are one 32-row tile.
template <int NT> struct VecF;
template <> struct VecF<2> { using type = float2; };
template <> struct VecF<4> { using type = float4; };

template <int NT>
__device__ __forceinline__ void vload(const float* p, float (&v)[NT]) {
  const typename VecF<NT>::type x = *reinterpret_cast<const typename VecF<NT>::type*>(p);
  if constexpr (NT == 2) { v[0] = x.x; v[1] = x.y; }
  else { v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w; }
}
template <int NT>
__device__ __forceinline__ void vstore(float* p, const float (&v)[NT]) {
  typename VecF<NT>::type x;
  if constexpr (NT == 2) { x.x = v[0]; x.y = v[1]; }
  else { x.x = v[0]; x.y = v[1]; x.z = v[2]; x.w = v[3]; }
  *reinterpret_cast<typename VecF<NT>::type*>(p) = x;
}

// HBM bounds it.  The rows that are added (ADD) and the pre-activations (AUX) are
// loaded eight at a time, the first before the products and the others one batch
// ahead of the stores.  One row's load at a time between the stores took 135 us for
// a forward layer of 32^3, batch 32 (403 MB), and 151 us for a backward one (537
// MB); this takes 95 (4.3 TB/s) and 110 us (4.9 TB/s).  For width 32, two voxels per
// lane and three waves per SIMD (with both kinds of rows two, the third spills: 142
// us): with four voxels one wave fits, 125 and 138 us.
template <int KS, int NT, bool ADD, bool AUX>
__global__ __launch_bounds__(256, ADD && AUX ? 1 : 3) void k_pointwise(PwArgs a) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  constexpr int BV = 32 * NT;   // voxels per wave block
  constexpr int GE = 8, NG = 16 / GE;   // rows loaded together
  typedef float VN __attribute__((ext_vector_type(NT)));
  const long long V = a.V;
  const long long blocks = (long long)a.B * (V / BV);
  const bf16x8* w8 = reinterpret_cast<const bf16x8*>(a.w);
  for (long long t = (long long)blockIdx.x * 4 + wave; t < blocks; t += (long long)gridDim.x * 4) {
    const int b = int(t / (V / BV));
    const long long v = (t % (V / BV)) * BV + NT * col;
    bf16x8 bop[KS][NT];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int i = s * 16 + half * 8 + j;
        float x[NT];
#pragma unroll
        for (int k = 0; k < NT; ++k) x[k] = 0.0f;
        if (i < a.I) vload<NT>(a.in + ((long long)b * a.I + i) * V + v, x);
#pragma unroll
        for (int k = 0; k < NT; ++k) bop[s][k][j] = (__bf16)x[k];
      }
    }
    // (a single round of kWidth channels: written straight on, the rows' addresses are
    // kept for all sixteen and the registers spill, 107 us for 95)
    for (int ot = 0; ot < a.opad / 32; ++ot) {
      // row of accumulator entry e; rows past the last one load the last one
      auto row = [&](int e) { return ot * 32 + 8 * (e / 4) + 4 * half + (e % 4); };
      VN ad[2][GE], ax[2][GE];
      auto fetch = [&](int g) {
#pragma unroll
        for (int k = 0; k < GE; ++k) {
          const int o = row(g * GE + k);
          const long long idx = ((long long)b * a.O + (o < a.O ? o : a.O - 1)) * V + v;
          if constexpr (ADD) ad[g & 1][k] = *reinterpret_cast<const VN*>(a.add + idx);
          if constexpr (AUX) ax[g & 1][k] = *reinterpret_cast<const VN*>(a.aux + idx);
        }
      };
      fetch(0);
      f32x16 acc[NT];
#pragma unroll
      for (int k = 0; k < NT; ++k) acc[k] = f32x16{0};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const bf16x8 aop = w8[((long long)(ot * 32 + col) * a.ipad + s * 16 + half * 8) / 8];
#pragma unroll
        for (int k = 0; k < NT; ++k) acc[k] = mfma(aop, bop[s][k], acc[k]);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        if (e % GE == 0 && e / GE + 1 < NG) {
          fetch(e / GE + 1);
          __builtin_amdgcn_sched_barrier(0);
        }
        const int o = row(e);
        if (o >= a.O) continue;
        const long long idx = ((long long)b * a.O + o) * V + v;
        float val[NT];
#pragma unroll
        for (int k = 0; k < NT; ++k) val[k] = acc[k][e];
        if (a.bias) {
          const float bo = a.bias[o];
#pragma unroll
          for (int k = 0; k < NT; ++k) val[k] += bo;
        }
        if constexpr (ADD) {
#pragma unroll
          for (int k = 0; k < NT; ++k) val[k] += ad[(e / GE) & 1][e % GE][k];
        }
        if constexpr (AUX) {
#pragma unroll
          for (int k = 0; k < NT; ++k) val[k] *= gelu_grad(ax[(e / GE) & 1][e % GE][k]);
        }
        if (a.out) vstore<NT>(a.out + idx, val);
        if (a.out_act) {
          float g[NT];
#pragma unroll
          for (int k = 0; k < NT; ++k) g[k] = gelu(val[k]);
          vstore<NT>(a.out_act + idx, g);
        }
      }
    }
  }
}

// lift: 16 or 32 padded input channels, nothing added; hidden layers: 32, the modes'
// part added, backward times GELU' of the layer before it (if there is one)
hipError_t launch_pointwise(const PwArgs& a, hipStream_t s) {
  const bool wide = a.ipad == 32;
  if ((a.ipad != 16 && !wide) || a.O != kWidth || a.opad != kWidth || a.V % 128 || (a.add && !wide) || (a.aux && !a.add))
    return hipErrorInvalidValue;
  const int nt = wide ? 2 : 4;
  const long long nblk = (long long)a.B * (a.V / (32 * nt));
  long long blocks = (nblk + 3) / 4;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  const dim3 g((unsigned)blocks);
  if (!wide) hipLaunchKernelGGL((k_pointwise<1, 4, false, false>), g, 256, 0, s, a);
  else if (a.aux) hipLaunchKernelGGL((k_pointwise<2, 2, true, true>), g, 256, 0, s, a);
  else if (a.add) hipLaunchKernelGGL((k_pointwise<2, 2, true, false>), g, 256, 0, s, a);
  else hipLaunchKernelGGL((k_pointwise<2, 2, false, false>), g, 256, 0, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// pointwise weight gradient: MFMA over 16-voxel chunks, per-block partials
// ---------------------------------------------------------------------------
// four workgroups to a CU: with one, a wave per SIMD, the loads' latency bound
// the width's products (94 us per layer at 32^3, batch 32)
constexpr int kWgBlocks = 1024;
int wgrad_blocks(int B, long long V) {
  const long long chunks = (long long)B * (V / 16);
  long long nb = (chunks + 3) / 4;
  return (int)(nb < kWgBlocks ? (nb < 1 ? 1 : nb) : kWgBlocks);
}

__global__ __launch_bounds__(256) void k_wgrad(WgArgs a) {
  __shared__ float red[4][1024 + 32];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int half = lane >> 5, row = lane & 31;
  const long long V = a.V;
  const long long chunks = (long long)a.B * (V / 16);
  f32x16 acc = f32x16{0};
  float bsum = 0.0f;
  for (long long c = (long long)blockIdx.x * 4 + wave; c < chunks; c += (long long)gridDim.x * 4) {
    const int b = int(c / (V / 16));
    const long long v0 = (c % (V / 16)) * 16 + half * 8;
    // eight consecutive voxels per lane: two 16-byte loads per operand row
    auto load8 = [&](const float* src, bool ok, float (&x)[8]) {
      float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
      if (ok) {
        lo = reinterpret_cast<const float4*>(src)[0];
        hi = reinterpret_cast<const float4*>(src)[1];
      }
      x[0] = lo.x; x[1] = lo.y; x[2] = lo.z; x[3] = lo.w;
      x[4] = hi.x; x[5] = hi.y; x[6] = hi.z; x[7] = hi.w;
    };
    bf16x8 aop, bop;
    float x[8];
    load8(a.h + ((long long)b * a.I + (row < a.I ? row : 0)) * V + v0, row < a.I, x);
#pragma unroll
    for (int j = 0; j < 8; ++j) bop[j] = (__bf16)x[j];
    load8(a.g + ((long long)b * a.O + (row < a.O ? row : 0)) * V + v0, row < a.O, x);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      bsum += x[j];
      aop[j] = (__bf16)x[j];
    }
    acc = mfma(aop, bop, acc);
  }
  // fixed-order sum of the four waves
  float* part = a.part + (size_t)blockIdx.x * (32 * 32 + 32);
#pragma unroll
  for (int e = 0; e < 16; ++e) red[wave][e * 64 + lane] = acc[e];
  // bias partial: lanes l and l + 32 hold the two halves of row l % 32
  if (half == 0) red[wave][1024 + row] = bsum;
  __syncthreads();
  if (half == 1) red[wave][1024 + row] += bsum;
  __syncthreads();
  for (int k = threadIdx.x; k < 1024; k += 256) {
    const float s = red[0][k] + red[1][k] + red[2][k] + red[3][k];
    const int e = k / 64, l = k % 64;
    part[(8 * (e / 4) + 4 * (l / 32) + (e % 4)) * 32 + (l & 31)] = s;
  }
  if (threadIdx.x < 32)
    part[1024 + threadIdx.x] = red[0][1024 + threadIdx.x] + red[1][1024 + threadIdx.x] + red[2][1024 + threadIdx.x] +
                               red[3][1024 + threadIdx.x];
}

// Fixed-order sum of the per-block partials: a workgroup covers 16 consecutive
// packed outputs, its 16 groups of lanes sum interleaved sixteenths of the
// partials with eight loads in flight, and the sixteenths are added in order.
// (64 outputs and quarters, one load at a time, took 24 us.)
__global__ __launch_bounds__(NTB) void k_wgrad_reduce(const float* __restrict__ part, int nblk, int O, int I,
                                                      int opad, int ipad, float* __restrict__ gw,
                                                      float* __restrict__ gb) {
  constexpr int U = 8;
  __shared__ float red[16][17];
  const int n = O * I + O;
  const size_t stride = (size_t)opad * ipad + opad;
  const int k = blockIdx.x * 16 + (threadIdx.x & 15);
  const int q = threadIdx.x >> 4;
  float s = 0.0f;
  if (k < n) {
    const float* src = part + ((k < O * I) ? (k / I) * ipad + (k % I) : opad * ipad + (k - O * I));
    for (int blk = q; blk < nblk; blk += 16 * U) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = (blk + 16 * u < nblk) ? src[(blk + 16 * u) * stride] : 0.0f;
#pragma unroll
      for (int u = 0; u < U; ++u) s += v[u];
    }
  }
  red[q][threadIdx.x & 15] = s;
  __syncthreads();
  if (q == 0 && k < n) {
    float t = 0.0f;
    for (int r = 0; r < 16; ++r) t += red[r][threadIdx.x];
    if (k < O * I) gw[k] = t;
    else gb[k - O * I] = t;
  }
}

static hipError_t launch_wgrad_reduce(const float* part, int nblk, int O, int I, int opad, int ipad, float* gw,
                                      float* gb, hipStream_t s) {
  const int n = O * I + O;
  hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)((n + 15) / 16)), NTB, 0, s, part, nblk, O, I, opad, ipad, gw, gb);
  return hipGetLastError();
}

hipError_t launch_wgrad(const WgArgs& a, float* gw, float* gb, hipStream_t s) {
  if (a.V % 16 || a.O > 32 || a.I > 32) return hipErrorInvalidValue;   // the width's layers: lift and hidden
  hipLaunchKernelGGL(k_wgrad, dim3((unsigned)a.nblk), 256, 0, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_wgrad_reduce(a.part, a.nblk, a.O, a.I, 32, 32, gw, gb, s);
}

// ---------------------------------------------------------------------------
// projection: hidden layer of `hidden` channels with GELU, then the output layer
// ---------------------------------------------------------------------------
// The accumulator tile of a 32-channel product has rows 8 q + 4 half + 0..3 in
// a lane's registers 4 q + 0..3; as the B operand of the next product the lane
// needs rows 16 s + 8 half + 0..7.  Exchanging the upper half-wave's group 2 s
// with the lower one's group 2 s + 1 gives exactly that, so a hidden tile goes
// from one product into the next without LDS.
__device__ __forceinline__ unsigned pack2(float a, float b) {
  union { unsigned short h[2]; unsigned u; } p;
  const __bf16 x = (__bf16)a, y = (__bf16)b;
  p.h[0] = __builtin_bit_cast(unsigned short, x);
  p.h[1] = __builtin_bit_cast(unsigned short, y);
  return p.u;
}
// B operands s = 0, 1 of a C-layout tile, its entries packed in pairs
__device__ __forceinline__ void as_operand(const unsigned (&pk)[8], bf16x8 (&op)[2]) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    union { unsigned u[4]; bf16x8 b; } r;
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const auto x = __builtin_amdgcn_permlane32_swap(pk[4 * s + d], pk[4 * s + 2 + d], false, false);
      r.u[d] = x[0];
      r.u[2 + d] = x[1];
    }
    op[s] = r.b;
  }
}

// y = W2 gelu(W1 h + b1) + b2; the hidden activations never leave registers
// (through HBM they were 1.6 GB per batch of 32 at 32^3 and 128 channels: 364 +
// 179 us for the two layers, 140 now).  Bound by the error functions: one per
// hidden channel and voxel.
__global__ __launch_bounds__(256) void k_project(ProjArgs a) {
  constexpr int NT = 2;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, col = lane & 31;
  constexpr int BV = 32 * NT;
  const long long V = a.V, blocks = (long long)a.B * (V / BV);
  const bf16x8* w1 = reinterpret_cast<const bf16x8*>(a.w1);
  const bf16x8* w2 = reinterpret_cast<const bf16x8*>(a.w2);
  for (long long t = (long long)blockIdx.x * 4 + wave; t < blocks; t += (long long)gridDim.x * 4) {
    const int b = int(t / (V / BV));
    const unsigned v = (unsigned)(t % (V / BV)) * BV + NT * col, Vu = (unsigned)V;
    const float* hb = a.h + (long long)b * 32 * V;
    float* yb = a.y + (long long)b * a.O * V;
    bf16x8 bop[2][NT];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float x[NT];
        vload<NT>(hb + ((s * 16 + half * 8 + j) * Vu + v), x);
#pragma unroll
        for (int k = 0; k < NT; ++k) bop[s][k][j] = (__bf16)x[k];
      }
    f32x16 acc2[NT];
#pragma unroll
    for (int k = 0; k < NT; ++k) acc2[k] = f32x16{0};
    for (int ot = 0; ot < a.hidden / 32; ++ot) {
      f32x16 acc[NT];
#pragma unroll
      for (int k = 0; k < NT; ++k) acc[k] = f32x16{0};
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const bf16x8 aop = w1[((ot * 32 + col) * 32 + s * 16 + half * 8) / 8];
#pragma unroll
        for (int k = 0; k < NT; ++k) acc[k] = mfma(aop, bop[s][k], acc[k]);
      }
      unsigned pk[NT][8];
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        const float b0 = a.b1[ot * 32 + 8 * (e / 4) + 4 * half + (e % 4)];
        const float b1 = a.b1[ot * 32 + 8 * (e / 4) + 4 * half + (e % 4) + 1];
#pragma unroll
        for (int k = 0; k < NT; ++k) pk[k][e / 2] = pack2(gelu(acc[k][e] + b0), gelu(acc[k][e + 1] + b1));
        __builtin_amdgcn_sched_barrier(0);   // few error functions at a time
      }
      bf16x8 aop2[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) aop2[s] = w2[(col * a.hidden + (ot * 2 + s) * 16 + half * 8) / 8];
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        bf16x8 op[2];
        as_operand(pk[k], op);
#pragma unroll
        for (int s = 0; s < 2; ++s) acc2[k] = mfma(aop2[s], op[s], acc2[k]);
      }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int o = 8 * (e / 4) + 4 * half + (e % 4);
      if (o >= a.O) continue;
      const float bo = a.b2[o];
      float val[NT];
#pragma unroll
      for (int k = 0; k < NT; ++k) val[k] = acc2[k][e] + bo;
      vstore<NT>(yb + (o * Vu + v), val);
    }
  }
}

hipError_t launch_project(const ProjArgs& a, hipStream_t s) {
  if (a.hidden % 32 || a.hidden < 32 || a.O > 32 || a.V % 64) return hipErrorInvalidValue;
  long long blocks = ((long long)a.B * (a.V / 64) + 3) / 4;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_project, dim3((unsigned)blocks), 256, 0, s, a);
  return hipGetLastError();
}

// Its backward pass, everything from h and dy: the hidden activations are
// formed again (the same products and roundings as forward), then per tile of 32
// voxels
//   dz = (W2^T dy) gelu'(p), dh = W1^T dz, gW2 += dy z^T, gW1 += dz h^T.
// Wave w of a workgroup owns hidden channels 32 w .. 32 w + 31: its two weight
// gradient tiles stay in accumulators over all voxels, with z and dz through a
// wave-private LDS tile for the products over voxels, and its dz goes to the
// others as operands through LDS.  dh sums over the hidden channels in their
// order, so one wave does a voxel tile's whole chain, each wave another tile.
// One erf and one exp per hidden channel and voxel bound it.  Before, the hidden
// layer's pre-activations, activations and gradients went through HBM over five
// kernels (327 + 239 + 230 + 213 us per batch of 32 at 32^3, 128 channels; 530
// now); with every hidden tile in one wave the accumulators left one wave per
// SIMD (953 us), without the next tile in flight it took 682.
constexpr int kPjPitch = 40;                    // bf16 row of an LDS tile
constexpr int kPjTile = 32 * kPjPitch;
constexpr int proj_tiles(int W) { return W < 4 ? W : 4; }   // voxel tiles of a workgroup
template <int W>
__global__ __launch_bounds__(64 * W, 2) void k_project_bwd(ProjBwdArgs a) {
  constexpr int NV = proj_tiles(W);
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, col = lane & 31;
  bf16x8* ops = reinterpret_cast<bf16x8*>(smem);               // [NV][2 W][64]: dz as B operands
  __bf16* zt = reinterpret_cast<__bf16*>(ops + NV * 2 * W * 64) + wave * 2 * kPjTile;   // [channel][voxel]
  __bf16* dt = zt + kPjTile;
  const long long V = a.V, groups = (long long)a.B * (V / 32) / NV;
  const int kso = a.opad16 / 16;                // k steps over the output channels (1 or 2)
  const unsigned Vu = (unsigned)V;
  f32x16 g1 = f32x16{0}, g2 = f32x16{0};
  float s1[16], s2 = 0.0f;
#pragma unroll
  for (int e = 0; e < 16; ++e) s1[e] = 0.0f;
  // channel rows of a voxel tile, one voxel per lane: the next tile's are in
  // flight while this one's error functions run
  float hn[2][8], yn[2][8];
  auto fetch = [&](long long t) {
    const int b = int(t / (V / 32));
    const unsigned v = (unsigned)(t % (V / 32)) * 32 + col;
    const float* hb = a.h + (long long)b * 32 * V;
    const float* yb = a.dy + (long long)b * a.O * V;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int c = s * 16 + half * 8 + j;
        hn[s][j] = hb[c * Vu + v];
        yn[s][j] = (s < kso && c < a.O) ? yb[c * Vu + v] : 0.0f;
      }
  };
  if ((long long)blockIdx.x < groups) fetch((long long)blockIdx.x * NV);
  for (long long gr = blockIdx.x; gr < groups; gr += gridDim.x) {
    const long long t0 = gr * NV;               // V / 32 is a multiple of NV: one sample per group
    const int b = int(t0 / (V / 32));
    const unsigned vg = (unsigned)(t0 % (V / 32)) * 32;
    const float* hb = a.h + (long long)b * 32 * V;
    const float* yb = a.dy + (long long)b * a.O * V;
#pragma unroll 1
    for (int i = 0; i < NV; ++i) {
      const unsigned v0 = vg + 32 * i;
      bf16x8 hop[2], yop[2];                    // h and dy as B operands (channel rows, voxel columns)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          hop[s][j] = (__bf16)hn[s][j];
          yop[s][j] = (__bf16)yn[s][j];
        }
      // dy and h as [channel][voxel] rows, for the products over voxels
      bf16x8 hw[2], yw[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const unsigned vr = v0 + s * 16 + half * 8;
        const f32x4* hr = reinterpret_cast<const f32x4*>(hb + (col * Vu + vr));
        const f32x4* yr = reinterpret_cast<const f32x4*>(yb + ((col < a.O ? col : 0) * Vu + vr));
        const f32x4 h0 = hr[0], h1 = hr[1];
        f32x4 y0 = yr[0], y1 = yr[1];
        if (col >= a.O) y0 = y1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          hw[s][j] = (__bf16)h0[j];
          hw[s][4 + j] = (__bf16)h1[j];
          yw[s][j] = (__bf16)y0[j];
          yw[s][4 + j] = (__bf16)y1[j];
          if (wave == 0) s2 += y0[j] + y1[j];
        }
      }
      {
        const long long nt = (i + 1 < NV) ? t0 + i + 1 : (gr + gridDim.x) * NV;
        if (nt < groups * NV) fetch(nt);
      }
      f32x16 p = f32x16{0}, d = f32x16{0};
      {
        const bf16x8* w1 = reinterpret_cast<const bf16x8*>(a.w1) + (wave * 32 + col) * 4 + half;
        const bf16x8* w2t = reinterpret_cast<const bf16x8*>(a.w2t) + (wave * 32 + col) * (2 * kso) + half;
        p = mfma(w1[0], hop[0], p);
        p = mfma(w1[2], hop[1], p);
        d = mfma(w2t[0], yop[0], d);
        if (kso > 1) d = mfma(w2t[2], yop[1], d);
      }
      unsigned pk[8];
      wave_order();                             // the last tile has been read
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        float dz[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int r = 8 * (e / 4) + 4 * half + (e % 4) + q;
          float z, gd;
          gelu_both(p[e + q] + a.b1[wave * 32 + r], z, gd);
          dz[q] = d[e + q] * gd;
          zt[r * kPjPitch + col] = (__bf16)z;
          dt[r * kPjPitch + col] = (__bf16)dz[q];
          s1[e + q] += dz[q];
        }
        pk[e / 2] = pack2(dz[0], dz[1]);
        __builtin_amdgcn_sched_barrier(0);      // few error functions at a time
      }
      bf16x8 op[2];
      as_operand(pk, op);
      ops[(i * 2 * W + 2 * wave) * 64 + lane] = op[0];
      ops[(i * 2 * W + 2 * wave + 1) * 64 + lane] = op[1];
      wave_order();
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        g2 = mfma(yw[s], *reinterpret_cast<const bf16x8*>(zt + col * kPjPitch + s * 16 + half * 8), g2);   // [o][hidden]
        g1 = mfma(*reinterpret_cast<const bf16x8*>(dt + col * kPjPitch + s * 16 + half * 8), hw[s], g1);   // [hidden][i]
      }
    }
    lsfft::lds_barrier();
    if (wave < NV) {
      const unsigned v = vg + 32 * wave + col;
      const bf16x8* w1t = reinterpret_cast<const bf16x8*>(a.w1t) + col * (4 * W) + half;
      f32x16 dh = f32x16{0};
#pragma unroll
      for (int s = 0; s < 2 * W; ++s) dh = mfma(w1t[2 * s], ops[(wave * 2 * W + s) * 64 + lane], dh);
      const float* pb = a.pre + (long long)b * 32 * V;
      float* ob = a.out + (long long)b * 32 * V;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const unsigned at = (8 * (e / 4) + 4 * half + (e % 4)) * Vu + v;
        ob[at] = dh[e] * gelu_grad(pb[at]);
      }
    }
    lsfft::lds_barrier();
  }
  // this wave's tiles into the block's partial slots; bias gradients summed over
  // the 32 voxel columns of each half-wave
  float* part2 = a.part2 + (size_t)blockIdx.x * (32 * a.hidden + 32);
  float* part1 = a.part1 + (size_t)blockIdx.x * (a.hidden * 32 + a.hidden);
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int r = 8 * (e / 4) + 4 * half + (e % 4);
    part1[(wave * 32 + r) * 32 + col] = g1[e];
    part2[r * a.hidden + wave * 32 + col] = g2[e];
    float t = s1[e];
#pragma unroll
    for (int m = 16; m > 0; m >>= 1) t += __shfl_xor(t, m, 64);
    if (col == 0) part1[a.hidden * 32 + wave * 32 + r] = t;
  }
  if (wave == 0) {
    s2 += __shfl_xor(s2, 32, 64);
    if (half == 0) part2[32 * a.hidden + col] = s2;
  }
}

// Two workgroups of four waves or more to a CU; below 128 hidden channels, where a
// workgroup has fewer waves, more of them: with 512 as well a batch of 32 at 32^3 took
// 848 us for 32 channels (286 now) and 637 for 64 (390).
int project_bwd_blocks(int B, long long V, int hidden) {
  const long long nb = (long long)B * (V / 32) / 4, most = 512 * std::max(1, 128 / hidden);
  return (int)(nb < most ? (nb < 1 ? 1 : nb) : most);
}

template <int W>
static hipError_t project_bwd(const ProjBwdArgs& a, int nblk, hipStream_t s) {
  constexpr size_t lds = (size_t)proj_tiles(W) * 2 * W * 64 * 16 + (size_t)W * 2 * kPjTile * 2;
  const hipError_t e = allow_lds(k_project_bwd<W>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_project_bwd<W>, dim3(nblk), 64 * W, lds, s, a);
  return hipGetLastError();
}

hipError_t launch_project_bwd(const ProjBwdArgs& a, float* gw1, float* gb1, float* gw2, float* gb2, hipStream_t s) {
  if (a.V % 128 || a.O > 32) return hipErrorInvalidValue;
  const int nblk = project_bwd_blocks(a.B, a.V, a.hidden);
  hipError_t e;
  switch (a.hidden) {
    case 32: e = project_bwd<1>(a, nblk, s); break;
    case 64: e = project_bwd<2>(a, nblk, s); break;
    case 128: e = project_bwd<4>(a, nblk, s); break;
    case 256: e = project_bwd<8>(a, nblk, s); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  e = launch_wgrad_reduce(a.part2, nblk, a.O, a.hidden, 32, a.hidden, gw2, gb2, s);
  if (e != hipSuccess) return e;
  return launch_wgrad_reduce(a.part1, nblk, a.hidden, 32, a.hidden, 32, gw1, gb1, s);
}

// ---------------------------------------------------------------------------
// per-mode complex products (one 256-thread block per eight modes)
// ---------------------------------------------------------------------------
// The modes are kept as md[m / 8][bc][m % 8] (see the transforms below), so a
// block reads and writes whole eight-mode groups as contiguous 16-byte runs,
// and each of its four waves multiplies two modes.  Operands go through LDS as
// bf16 planes, A as [row][k] and (mode 2) B transposed as [n][k], so every MFMA
// operand is one 16-byte LDS read; the weights of modes 0 and 1 are read from
// HBM straight into the operand registers.  Products leave through LDS in the
// group layout.  HBM bounds it: at 6,912 modes and batch 32, 57 MB in, 28 MB of
// weights, 57 MB out.
constexpr int kMg = 8;                          // modes per group
constexpr int kMixPitch = 32 + 8;               // bf16 plane row
constexpr int kMixPlane = 32 * kMixPitch + 16;  // plane of one mode
constexpr int kMixOut = kMg + 1;                // complex entries per bc of the staged products
constexpr int kMixBytes0 = 1024 * kMixOut * 8;  // modes 0 and 1 (covers the two A planes)
constexpr int kMixBytes2 = 4 * kMg * kMixPlane * 2;
static_assert(2 * kMg * kMixPlane * 2 <= kMixBytes0, "operand planes under the staged products");

template <int MODE>
__global__ __launch_bounds__(256) void k_modemix(const float2* __restrict__ x, const __hip_bfloat16* __restrict__ rb,
                                                 const float2* __restrict__ g, float* __restrict__ out, int nmodes,
                                                 int B) {
  extern __shared__ __align__(16) unsigned char smem[];
  __bf16* P = reinterpret_cast<__bf16*>(smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;
  const int grp = blockIdx.x;
  const size_t BC = (size_t)B * 32;
  const float4* x4 = reinterpret_cast<const float4*>(x + (size_t)grp * BC * kMg);
  const float4* g4 = reinterpret_cast<const float4*>(g + (MODE == 2 ? (size_t)grp * BC * kMg : 0));
  auto plane = [&](int which, int m) { return P + (which * kMg + m) * kMixPlane; };
  const int nbt = (B + 31) / 32;

  // weights of this wave's two modes as B operands:
  // B^T[n][k]: mode 0 -> R[k][n] (n = o, k = i); mode 1 -> conj R[n][k] (n = i, k = o)
  bf16x8 wr[MODE == 2 ? 1 : 2][2], wi[MODE == 2 ? 1 : 2][2];
  if constexpr (MODE != 2) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int m = grp * kMg + wave * 2 + q;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int k0 = s * 16 + half * 8;
        unsigned w[8];
        if (m < nmodes) {
          const unsigned* rm = reinterpret_cast<const unsigned*>(rb) + (size_t)m * 1024;   // (re, im) pairs
          if constexpr (MODE == 0) {
#pragma unroll
            for (int j = 0; j < 8; ++j) w[j] = rm[(k0 + j) * 32 + col];
          } else {
            const uint4 lo = reinterpret_cast<const uint4*>(rm + col * 32 + k0)[0];
            const uint4 hi = reinterpret_cast<const uint4*>(rm + col * 32 + k0)[1];
            w[0] = lo.x; w[1] = lo.y; w[2] = lo.z; w[3] = lo.w;
            w[4] = hi.x; w[5] = hi.y; w[6] = hi.z; w[7] = hi.w;
          }
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) w[j] = 0u;
        }
        union { unsigned short h[8]; bf16x8 v; } re, im;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          re.h[j] = (unsigned short)(w[j] & 0xffffu);
          im.h[j] = (unsigned short)((w[j] >> 16) ^ (MODE == 1 ? 0x8000u : 0u));   // conj: sign flipped
        }
        wr[q][s] = re.v;
        wi[q][s] = im.v;
      }
    }
  }

  f32x16 cr[2], ci[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    cr[q] = f32x16{0};
    ci[q] = f32x16{0};
  }
  for (int bt = 0; bt < nbt; ++bt) {
    if (bt > 0) __syncthreads();
    // 32 samples x 32 channels x 8 modes: thread t takes the mode pair t % 4
    // of bc = t / 4, t / 4 + 64, ...
    const int mp = tid & 3;
#pragma unroll
    for (int u0 = 0; u0 < 16; u0 += 4) {
      float4 v[4], w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int bc = (tid >> 2) + 64 * (u0 + u);
        const bool ok = bt * 32 + (bc >> 5) < B;
        v[u] = w[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ok) {
          v[u] = x4[((size_t)bt * 1024 + bc) * 4 + mp];
          if constexpr (MODE == 2) w[u] = g4[((size_t)bt * 1024 + bc) * 4 + mp];
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int bc = (tid >> 2) + 64 * (u0 + u);
        const int rr = bc >> 5, c = bc & 31;
        if constexpr (MODE != 2) {
          // A[row = b][k]: mode 0 x[b][i], mode 1 g[b][o] (passed in x)
          const int at = rr * kMixPitch + c;
          plane(0, 2 * mp)[at] = (__bf16)v[u].x;
          plane(1, 2 * mp)[at] = (__bf16)v[u].y;
          plane(0, 2 * mp + 1)[at] = (__bf16)v[u].z;
          plane(1, 2 * mp + 1)[at] = (__bf16)v[u].w;
        } else {
          // A[row = i][k = b] = conj x[b][i]; B^T[n = o][k = b] = g[b][o]
          const int at = c * kMixPitch + rr;
          plane(0, 2 * mp)[at] = (__bf16)v[u].x;
          plane(1, 2 * mp)[at] = (__bf16)(-v[u].y);
          plane(0, 2 * mp + 1)[at] = (__bf16)v[u].z;
          plane(1, 2 * mp + 1)[at] = (__bf16)(-v[u].w);
          plane(2, 2 * mp)[at] = (__bf16)w[u].x;
          plane(3, 2 * mp)[at] = (__bf16)w[u].y;
          plane(2, 2 * mp + 1)[at] = (__bf16)w[u].z;
          plane(3, 2 * mp + 1)[at] = (__bf16)w[u].w;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int m = wave * 2 + q;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int at = col * kMixPitch + s * 16 + half * 8;
        const bf16x8 ar = *reinterpret_cast<const bf16x8*>(plane(0, m) + at);
        const bf16x8 ai = *reinterpret_cast<const bf16x8*>(plane(1, m) + at);
        bf16x8 br, bi;
        if constexpr (MODE == 2) {
          br = *reinterpret_cast<const bf16x8*>(plane(2, m) + at);
          bi = *reinterpret_cast<const bf16x8*>(plane(3, m) + at);
        } else {
          br = wr[q][s];
          bi = wi[q][s];
        }
        cr[q] = mfma(ar, br, cr[q]);
        cr[q] = mfma(neg8(ai), bi, cr[q]);
        ci[q] = mfma(ar, bi, ci[q]);
        ci[q] = mfma(ai, br, ci[q]);
      }
    }
    if constexpr (MODE != 2) {
      __syncthreads();   // the planes have been read: the products replace them
      float2* so = reinterpret_cast<float2*>(smem);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int rr = 8 * (e / 4) + 4 * half + (e % 4);
          so[(rr * 32 + col) * kMixOut + wave * 2 + q] = make_float2(cr[q][e], ci[q][e]);
        }
        cr[q] = f32x16{0};
        ci[q] = f32x16{0};
      }
      __syncthreads();
      float4* o4 = reinterpret_cast<float4*>(reinterpret_cast<float2*>(out) + (size_t)grp * BC * kMg);
#pragma unroll 4
      for (int u = 0; u < 16; ++u) {
        const int bc = (tid >> 2) + 64 * u;
        if (bt * 32 + (bc >> 5) >= B) continue;
        const float2 p = so[bc * kMixOut + 2 * mp], r = so[bc * kMixOut + 2 * mp + 1];
        o4[((size_t)bt * 1024 + bc) * 4 + mp] = make_float4(p.x, p.y, r.x, r.y);
      }
    }
  }
  if constexpr (MODE == 2) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int m = grp * kMg + wave * 2 + q;
      if (m >= nmodes) continue;
      float2* om = reinterpret_cast<float2*>(out) + (size_t)m * 32 * 32;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int i = 8 * (e / 4) + 4 * half + (e % 4);
        om[i * 32 + col] = make_float2(cr[q][e], ci[q][e]);
      }
    }
  }
}

hipError_t launch_modemix(int mode, const float2* x, const __hip_bfloat16* r, const float2* g, float* out,
                          int nmodes, int B, hipStream_t s) {
  const dim3 grid((unsigned)((nmodes + kMg - 1) / kMg));
  hipError_t e;
  if (mode == 0) {
    if ((e = allow_lds(k_modemix<0>, kMixBytes0)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_modemix<0>, grid, 256, kMixBytes0, s, x, r, g, out, nmodes, B);
  } else if (mode == 1) {
    if ((e = allow_lds(k_modemix<1>, kMixBytes0)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_modemix<1>, grid, 256, kMixBytes0, s, x, r, g, out, nmodes, B);
  } else if (mode == 2) {
    if ((e = allow_lds(k_modemix<2>, kMixBytes2)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_modemix<2>, grid, 256, kMixBytes2, s, x, r, g, out, nmodes, B);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// truncated transforms: one cube of one (sample, channel) per workgroup
// ---------------------------------------------------------------------------
// All three axes of a cube in one launch, the truncated spectrum between the
// axes in LDS: a thread holds one pencil of N points in registers and runs the
// whole length-N Stockham transform there (the radices and operations of the
// solver's plans), so LDS only carries the kept entries from one axis to the
// next, in place.  One launch per axis through HBM moved 541 MB per batch of
// 32 at N = 32, M = 12 (45 + 31 + 38 us forward, 32 + 32 + 55 us inverse)
// where 191 MB are needed; a cube takes one launch of 62 us forward and 56
// inverse.  Registers allow two waves per SIMD, and the three phases' transforms
// (VALU) and their LDS exchange, one after the other, bound it.
//
// LDS entry (z, y or iy, kx) of the cube sits at z PP + y MP + kx: MP odd, so
// the lanes of the x phase (one row each) fall on different banks, and PP = M
// modulo 16, so that consecutive pencils of the y phase are consecutive across
// planes too.
//
//   h, out  [BC][z][y][x]                 real
//   md      [m / 8][BC][m % 8]            the kept modes m = iz P + iy M + kx,
//                                         P = 2 M^2, iy and iz in [0, 2M)
// Kept array index of FFT index k: k for k < M, k - n + 2M for k >= n - M.
template <int N> __device__ __forceinline__ constexpr int kslot(int k, int M) {
  return k < M ? k : (k >= N - M ? k - N + 2 * M : -1);
}
template <int N> constexpr int cube_threads() { return N * N < 512 ? N * N : 512; }

// a product rounded by itself, whatever is added to it next
__device__ __forceinline__ float scaled(float x, float c) {
#pragma clang fp contract(off)
  return x * c;
}

// The twiddles exp(-2 pi i k / N) that the second pass uses, in scalar
// registers for the whole kernel: left to the compiler they are vector loads
// inside every transform, whose waits also wait for the next cube's rows.
template <int N> struct RegTw {
  static constexpr int CNT = lsfft::Plan<N>::np == 1 ? 1 : (lsfft::Plan<N>::r1 - 1) * (N / lsfft::Plan<N>::r1 - 1) + 1;
  float r[CNT], i[CNT];
  __device__ __forceinline__ void load(const float2* __restrict__ tw) {
#pragma unroll
    for (int k = 0; k < CNT; ++k) {
      const float2 w = tw[k];
      r[k] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(w.x)));
      i[k] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(w.y)));
    }
  }
};

template <int N, int DIR> struct RegFft {
  using P = lsfft::Plan<N>;
  static_assert(P::np <= 2, "two-pass plans");
  // positions 0..N-1 in and out
  __device__ static __forceinline__ void run(float (&vr)[N], float (&vi)[N], const RegTw<N>& tw) {
    constexpr int R0 = P::r0, R1 = P::r1;
    if constexpr (P::np == 1) {
      lsfft::bfly<float, R0, DIR>(vr, vi);
    } else {
      float tr[N], ti[N];
#pragma unroll
      for (int j = 0; j < N / R0; ++j) {
        float ar[R0], ai[R0];
#pragma unroll
        for (int r = 0; r < R0; ++r) {
          ar[r] = vr[j + r * (N / R0)];
          ai[r] = vi[j + r * (N / R0)];
        }
        lsfft::bfly<float, R0, DIR>(ar, ai);
#pragma unroll
        for (int r = 0; r < R0; ++r) {
          tr[j * R0 + r] = ar[r];
          ti[j * R0 + r] = ai[r];
        }
      }
#pragma unroll
      for (int j = 0; j < N / R1; ++j) {
        float ar[R1], ai[R1];
#pragma unroll
        for (int r = 0; r < R1; ++r) {
          ar[r] = tr[j + r * (N / R1)];
          ai[r] = ti[j + r * (N / R1)];
        }
#pragma unroll
        for (int r = 1; r < R1; ++r) {
          const float br = tw.r[r * j], bi = (DIR < 0) ? tw.i[r * j] : -tw.i[r * j];
          // (rounded as the tile transforms round it, so the bits do not depend on
          // what the compiler contracts here)
          const float t = __builtin_fmaf(ar[r], br, -scaled(ai[r], bi));
          ai[r] = __builtin_fmaf(ai[r], br, scaled(ar[r], bi));
          ar[r] = t;
        }
        lsfft::bfly<float, R1, DIR>(ar, ai);
#pragma unroll
        for (int r = 0; r < R1; ++r) {
          vr[j + r * (N / R1)] = ar[r];
          vi[j + r * (N / R1)] = ai[r];
        }
      }
    }
  }
};

struct CubeArgs {
  int M, BC;
  int MP, PP;      // LDS pitches of a row and of a plane (complex entries)
  float s0, s1;    // scale of kx = 0 and of kx > 0
  const float2* tw;
};
__device__ __forceinline__ size_t md_at(int m, int bc, int BC) {
  return ((size_t)(m >> 3) * BC + bc) * kMg + (m & 7);
}
// Blocks of one XCD take consecutive cubes: their 64-byte runs of a mode group
// then meet in that XCD's L2.
__device__ __forceinline__ int cube_slot(int b, int G) {
  const int q = G / 8, r = G % 8, x = b % 8;
  return x * q + (x < r ? x : r) + b / 8;
}

// A wave's 64 rows between HBM and one row per lane, through a wave-private
// stretch of LDS (its own rows of the cube: no barrier), 16 entries at a time at
// a pitch of 20 words.  HBM sees 64-byte runs of four lanes; a row per lane
// straight from HBM touches 64 lines per access and keeps 64 KB of them open,
// twice the L1 (the inverse took 72 us per batch of 32 at N = 32 that way).
constexpr int kRowPitch = 20, kRowStage = 64 * kRowPitch * 4;   // words, bytes per wave
template <int N>
__device__ __forceinline__ void rows_fetch(const float* __restrict__ src, f32x4 (&v)[N / 4], int lane) {
  // piece i of 16 entries: rows (i % 4) * 16 + lane / 4, entries 16 (i / 4) + 4 (lane % 4)
#pragma unroll
  for (int i = 0; i < N / 4; ++i)
    v[i] = *reinterpret_cast<const f32x4*>(src + ((i & 3) * 16 + (lane >> 2)) * N + (i >> 2) * 16 + 4 * (lane & 3));
}
template <int N>
__device__ __forceinline__ void rows_spread(const f32x4 (&v)[N / 4], float (&row)[N], float* st, int lane) {
#pragma unroll
  for (int hh = 0; hh < N / 16; ++hh) {
    wave_order();
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<f32x4*>(st + (i * 16 + (lane >> 2)) * kRowPitch + 4 * (lane & 3)) = v[hh * 4 + i];
    wave_order();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(st + lane * kRowPitch + 4 * k);
      row[hh * 16 + 4 * k] = x.x;
      row[hh * 16 + 4 * k + 1] = x.y;
      row[hh * 16 + 4 * k + 2] = x.z;
      row[hh * 16 + 4 * k + 3] = x.w;
    }
  }
  wave_order();
}
template <int N>
__device__ __forceinline__ void rows_store(float* __restrict__ dst, const float (&row)[N], float* st, int lane) {
#pragma unroll
  for (int hh = 0; hh < N / 16; ++hh) {
    wave_order();
#pragma unroll
    for (int k = 0; k < 4; ++k)
      *reinterpret_cast<float4*>(st + lane * kRowPitch + 4 * k) =
          make_float4(row[hh * 16 + 4 * k], row[hh * 16 + 4 * k + 1], row[hh * 16 + 4 * k + 2], row[hh * 16 + 4 * k + 3]);
    wave_order();
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<float4*>(dst + (i * 16 + (lane >> 2)) * N + hh * 16 + 4 * (lane & 3)) =
          *reinterpret_cast<const float4*>(st + (i * 16 + (lane >> 2)) * kRowPitch + 4 * (lane & 3));
  }
  wave_order();
}

// h -> kept modes.  The next cube's rows are in flight during the y and z
// phases.
template <int N>
__global__ __launch_bounds__(cube_threads<N>()) void k_cube_fwd(const float* __restrict__ h, float2* __restrict__ md,
                                                                CubeArgs a) {
  constexpr int NT = cube_threads<N>(), RPT = N * N / NT;
  static_assert(RPT <= 2, "two rows per thread");
  extern __shared__ __align__(16) unsigned char smem[];
  float2* L = reinterpret_cast<float2*>(smem);
  RegTw<N> tw;
  tw.load(a.tw);
  const int M = a.M, P = 2 * M * M;
  constexpr bool STG = N >= 16;                       // 8-point rows go straight
  auto load = [&](int bc, int q, int wave, int lane, f32x4 (&v)[N / 4]) {
    const float* src = h + ((size_t)bc * N * N + wave * 64 + q * NT) * N;
    if constexpr (STG) {
      rows_fetch<N>(src, v, lane);
    } else {
#pragma unroll
      for (int k = 0; k < N / 4; ++k) v[k] = reinterpret_cast<const f32x4*>(src + lane * N)[k];
    }
  };
  int bc = cube_slot(blockIdx.x, gridDim.x);
  f32x4 in[RPT][N / 4];
  if (bc < a.BC) {
#pragma unroll
    for (int q = 0; q < RPT; ++q) load(bc, q, threadIdx.x >> 6, threadIdx.x & 63, in[q]);
  }
  for (; bc < a.BC; bc += gridDim.x) {
    // opaque: what follows from the thread's number is formed in every cube, not
    // kept in registers (and spilled) across all of them
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      float vr[N], vi[N];
#pragma unroll
      for (int k = 0; k < N; ++k) vi[k] = 0.0f;
      const int r0 = wave * 64 + q * NT;              // this wave's first row
      if constexpr (STG) {
        rows_spread<N>(in[q], vr, reinterpret_cast<float*>(L + (r0 / N) * a.PP), lane);
      } else {
#pragma unroll
        for (int k = 0; k < N / 4; ++k) {
          vr[4 * k] = in[q][k].x;
          vr[4 * k + 1] = in[q][k].y;
          vr[4 * k + 2] = in[q][k].z;
          vr[4 * k + 3] = in[q][k].w;
        }
      }
      RegFft<N, -1>::run(vr, vi, tw);
      // the upper half is formed too, as everywhere else: left out, its
      // partners' products have one use and are contracted into other roundings
#pragma unroll
      for (int k = N / 2; k < N; ++k) asm volatile("" ::"v"(vr[k]), "v"(vi[k]));
      const int r = tid + q * NT;
      float2* dst = L + (r / N) * a.PP + (r % N) * a.MP;
#pragma unroll
      for (int k = 0; k < N / 2; ++k)
        if (k < M) dst[k] = make_float2(vr[k], vi[k]);
      __builtin_amdgcn_sched_barrier(0);   // one row's transform at a time: two interleaved spill
    }
    lsfft::lds_barrier();
    if (bc + (int)gridDim.x < a.BC) {
#pragma unroll
      for (int q = 0; q < RPT; ++q) load(bc + gridDim.x, q, wave, lane, in[q]);
    }
    if (tid < N * M) {
      const int z = tid / M, kx = tid - z * M;
      float2* p = L + z * a.PP + kx;
      float vr[N], vi[N];
#pragma unroll
      for (int y = 0; y < N; ++y) {
        const float2 v = p[y * a.MP];
        vr[y] = v.x;
        vi[y] = v.y;
      }
      RegFft<N, -1>::run(vr, vi, tw);
#pragma unroll
      for (int y = 0; y < N; ++y) {
        const int iy = kslot<N>(y, M);
        if (iy >= 0) p[iy * a.MP] = make_float2(vr[y], vi[y]);
      }
    }
    lsfft::lds_barrier();
    if (tid < P) {
      const int iy = tid / M, kx = tid - iy * M;
      const float2* p = L + iy * a.MP + kx;
      float vr[N], vi[N];
#pragma unroll
      for (int z = 0; z < N; ++z) {
        const float2 v = p[z * a.PP];
        vr[z] = v.x;
        vi[z] = v.y;
      }
      RegFft<N, -1>::run(vr, vi, tw);
      const float sc = (kx == 0) ? a.s0 : a.s1;
#pragma unroll
      for (int z = 0; z < N; ++z) {
        const int iz = kslot<N>(z, M);
        if (iz >= 0) md[md_at(iz * P + tid, bc, a.BC)] = make_float2(vr[z] * sc, vi[z] * sc);
      }
    }
    lsfft::lds_barrier();
  }
}

// kept modes -> out[x] = sum over kx of c(kx) Re(. e^{+i kx x}), c = s0, s1.
// The next cube's modes are in flight during the y and x phases.
template <int N>
__global__ __launch_bounds__(cube_threads<N>()) void k_cube_inv(const float2* __restrict__ md, float* __restrict__ out,
                                                                CubeArgs a) {
  constexpr int NT = cube_threads<N>(), RPT = N * N / NT;
  extern __shared__ __align__(16) unsigned char smem[];
  float2* L = reinterpret_cast<float2*>(smem);
  RegTw<N> tw;
  tw.load(a.tw);
  const int tid0 = threadIdx.x, M = a.M, P = 2 * M * M;
  float zr[N], zi[N];
  auto load = [&](int bc, int tid) {
#pragma unroll
    for (int z = 0; z < N; ++z) {
      const int iz = kslot<N>(z, M);
      float2 v = make_float2(0.0f, 0.0f);
      if (iz >= 0 && tid < P) v = md[md_at(iz * P + tid, bc, a.BC)];
      zr[z] = v.x;
      zi[z] = v.y;
    }
  };
  int bc = cube_slot(blockIdx.x, gridDim.x);
  if (bc < a.BC) load(bc, tid0);
  for (; bc < a.BC; bc += gridDim.x) {
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    if (tid < P) {
      RegFft<N, 1>::run(zr, zi, tw);
      const int iy = tid / M, kx = tid - iy * M;
      float2* p = L + iy * a.MP + kx;
#pragma unroll
      for (int z = 0; z < N; ++z) p[z * a.PP] = make_float2(zr[z], zi[z]);
    }
    lsfft::lds_barrier();
    if (bc + (int)gridDim.x < a.BC) load(bc + gridDim.x, tid);
    if (tid < N * M) {
      const int z = tid / M, kx = tid - z * M;
      float2* p = L + z * a.PP + kx;
      float vr[N], vi[N];
#pragma unroll
      for (int y = 0; y < N; ++y) {
        const int iy = kslot<N>(y, M);
        float2 v = make_float2(0.0f, 0.0f);
        if (iy >= 0) v = p[iy * a.MP];
        vr[y] = v.x;
        vi[y] = v.y;
      }
      RegFft<N, 1>::run(vr, vi, tw);
#pragma unroll
      for (int y = 0; y < N; ++y) p[y * a.MP] = make_float2(vr[y], vi[y]);
    }
    lsfft::lds_barrier();
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const int r = tid + q * NT;
      const float2* src = L + (r / N) * a.PP + (r % N) * a.MP;
      float vr[N], vi[N];
#pragma unroll
      for (int k = 0; k < N; ++k) {
        vr[k] = 0.0f;
        vi[k] = 0.0f;
        if (k < N / 2 && k < M) {
          const float2 v = src[k];
          const float c = (k == 0) ? a.s0 : a.s1;
          vr[k] = scaled(v.x, c);
          vi[k] = scaled(v.y, c);
        }
      }
      RegFft<N, 1>::run(vr, vi, tw);
      if constexpr (N >= 16) {
        const int r0 = (tid & ~63) + q * NT;          // this wave's first row
        rows_store<N>(out + ((size_t)bc * N * N + r0) * N, vr, reinterpret_cast<float*>(L + (r0 / N) * a.PP), tid & 63);
      } else {
        float4* dst = reinterpret_cast<float4*>(out + ((size_t)bc * N * N + r) * N);
#pragma unroll
        for (int k = 0; k < N / 4; ++k) dst[k] = make_float4(vr[4 * k], vr[4 * k + 1], vr[4 * k + 2], vr[4 * k + 3]);
      }
    }
    lsfft::lds_barrier();
  }
}

template <int N>
static hipError_t cube_n(bool fwd, int M, int BC, const float* h, const float2* md_in, float2* md_out, float* out,
                         float s0, float s1, const float2* tw, hipStream_t s) {
  CubeArgs a{};
  a.M = M;
  a.BC = BC;
  a.MP = M | 1;
  // a plane holds its rows and its share of a wave's row staging
  const int need = std::max(N * a.MP, N >= 16 ? kRowStage * N / (64 * 8) : 0);
  a.PP = need + ((M - need) % 16 + 16) % 16;
  a.s0 = s0;
  a.s1 = s1;
  a.tw = tw;
  const size_t lds = (size_t)N * a.PP * sizeof(float2);
  if (lds > (size_t)lsfft::kMaxDynamicLds) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)(BC < 256 * (N == 32 ? 1 : 4) ? BC : 256 * (N == 32 ? 1 : 4));
  hipError_t e = fwd ? allow_lds(k_cube_fwd<N>, lds) : allow_lds(k_cube_inv<N>, lds);
  if (e != hipSuccess) return e;
  if (fwd) hipLaunchKernelGGL(k_cube_fwd<N>, dim3(grid), cube_threads<N>(), lds, s, h, md_out, a);
  else hipLaunchKernelGGL(k_cube_inv<N>, dim3(grid), cube_threads<N>(), lds, s, md_in, out, a);
  return hipGetLastError();
}

static hipError_t cube(bool fwd, int n, int M, int BC, const float* h, const float2* md_in, float2* md_out,
                       float* out, float s0, float s1, const float2* tw, hipStream_t s) {
  if (M < 1 || 2 * M > n || BC < 1) return hipErrorInvalidValue;
  switch (n) {
    case 8: return cube_n<8>(fwd, M, BC, h, md_in, md_out, out, s0, s1, tw, s);
    case 16: return cube_n<16>(fwd, M, BC, h, md_in, md_out, out, s0, s1, tw, s);
    case 32: return cube_n<32>(fwd, M, BC, h, md_in, md_out, out, s0, s1, tw, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_dft_forward(int n, int M, int BC, const float* h, float2* md, float sc0, float sc1,
                              const float2* tw, hipStream_t s) {
  return cube(true, n, M, BC, h, nullptr, md, nullptr, sc0, sc1, tw, s);
}

hipError_t launch_dft_inverse(int n, int M, int BC, const float2* md, float* out, float c0, float c1,
                              const float2* tw, hipStream_t s) {
  return cube(false, n, M, BC, nullptr, md, nullptr, out, c0, c1, tw, s);
}

// ---------------------------------------------------------------------------
// loss, Adam, casts
// ---------------------------------------------------------------------------
__device__ double block_sum_d(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < NTB / 64; ++k) s += red[k];
  return s;
}

// part[b][chunk][2] = (sum (y - t)^2, sum t^2) over one chunk of sample b
__global__ __launch_bounds__(NTB) void k_loss_part(const float* __restrict__ y, const float* __restrict__ t,
                                                   long long per, int nchunk, double* __restrict__ part) {
  __shared__ double red[NTB / 64];
  const int b = blockIdx.y, c = blockIdx.x;
  const long long len = (per + nchunk - 1) / nchunk;
  const long long lo = c * len, hi = (lo + len < per) ? lo + len : per;
  double e = 0.0, n = 0.0;
  for (long long k = lo + threadIdx.x; k < hi; k += NTB) {
    const double d = (double)y[b * per + k] - (double)t[b * per + k];
    const double tv = (double)t[b * per + k];
    e += d * d;
    n += tv * tv;
  }
  e = block_sum_d(e, red);
  n = block_sum_d(n, red);
  if (threadIdx.x == 0) {
    part[((size_t)b * nchunk + c) * 2] = e;
    part[((size_t)b * nchunk + c) * 2 + 1] = n;
  }
}

// per-sample coefficients 1 / (||e_b|| ||t_b|| B) and the mean loss (one
// block; a thread per sample, then a fixed-order sum)
__global__ __launch_bounds__(NTB) void k_loss_final(const double* __restrict__ part, int B, int nchunk,
                                                    double* __restrict__ coef, double* __restrict__ loss) {
  __shared__ double red[NTB];
  double acc = 0.0;
  for (int b = threadIdx.x; b < B; b += NTB) {
    double e = 0.0, n = 0.0;
    for (int c = 0; c < nchunk; ++c) {
      e += part[((size_t)b * nchunk + c) * 2];
      n += part[((size_t)b * nchunk + c) * 2 + 1];
    }
    const double en = sqrt(e), tn = sqrt(n);
    acc += en / tn;
    coef[b] = 1.0 / (fmax(en, 1e-300) * tn * (double)B);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int k = 0; k < NTB; ++k) s += red[k];
    *loss = s / (double)B;
  }
}

__global__ __launch_bounds__(NTB) void k_loss_grad(const float* __restrict__ y, const float* __restrict__ t,
                                                   const double* __restrict__ coef, float* __restrict__ dy, int B,
                                                   long long per) {
  const long long n = (long long)B * per;
  for (long long k = (long long)blockIdx.x * NTB + threadIdx.x; k < n; k += (long long)gridDim.x * NTB)
    dy[k] = (float)(((double)y[k] - (double)t[k]) * coef[k / per]);
}

hipError_t launch_loss(const float* y, const float* t, float* dy, int B, long long per_sample, double* part,
                       int nchunk, double* loss_dev, hipStream_t s) {
  double* coef = part + (size_t)B * nchunk * 2;
  hipLaunchKernelGGL(k_loss_part, dim3((unsigned)nchunk, (unsigned)B), NTB, 0, s, y, t, per_sample, nchunk, part);
  hipLaunchKernelGGL(k_loss_final, dim3(1), NTB, 0, s, part, B, nchunk, coef, loss_dev);
  long long blocks = ((long long)B * per_sample + NTB - 1) / NTB;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_loss_grad, dim3((unsigned)blocks), NTB, 0, s, y, t, coef, dy, B, per_sample);
  return hipGetLastError();
}

__global__ __launch_bounds__(NTB) void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                                              float* __restrict__ v, long long n, float lr, float b1, float b2,
                                              float eps, float bc1, float bc2) {
  for (long long k = (long long)blockIdx.x * NTB + threadIdx.x; k < n; k += (long long)gridDim.x * NTB) {
    const float gk = g[k];
    const float mk = b1 * m[k] + (1.0f - b1) * gk;
    const float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    p[k] -= lr * (mk / bc1) / (sqrtf(vk / bc2) + eps);
  }
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, long long n, float lr, float b1, float b2,
                       float eps, float bc1, float bc2, hipStream_t s) {
  long long blocks = (n + NTB - 1) / NTB;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_adam, dim3((unsigned)blocks), NTB, 0, s, p, g, m, v, n, lr, b1, b2, eps, bc1, bc2);
  return hipGetLastError();
}

__global__ __launch_bounds__(NTB) void k_cast_pad(const float* __restrict__ src, int rows, int cols, long long sr,
                                                  long long sc, __hip_bfloat16* __restrict__ dst, int drows, int dcols) {
  __bf16* d = reinterpret_cast<__bf16*>(dst);
  const long long n = (long long)drows * dcols;
  for (long long k = (long long)blockIdx.x * NTB + threadIdx.x; k < n; k += (long long)gridDim.x * NTB) {
    const int r = int(k / dcols), c = int(k % dcols);
    d[k] = (__bf16)((r < rows && c < cols) ? src[r * sr + c * sc] : 0.0f);
  }
}

hipError_t launch_cast_pad(const float* src, int rows, int cols, long long sr, long long sc, __hip_bfloat16* dst,
                           int drows, int dcols, hipStream_t s) {
  long long blocks = ((long long)drows * dcols + NTB - 1) / NTB;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_cast_pad, dim3((unsigned)blocks), NTB, 0, s, src, rows, cols, sr, sc, dst, drows, dcols);
  return hipGetLastError();
}

__global__ __launch_bounds__(NTB) void k_cast(const float* __restrict__ src, __hip_bfloat16* __restrict__ dst,
                                              long long n) {
  __bf16* d = reinterpret_cast<__bf16*>(dst);
  for (long long k = (long long)blockIdx.x * NTB + threadIdx.x; k < n; k += (long long)gridDim.x * NTB)
    d[k] = (__bf16)src[k];
}

hipError_t launch_cast(const float* src, __hip_bfloat16* dst, long long n, hipStream_t s) {
  long long blocks = (n + NTB - 1) / NTB;
  if (blocks > 8192) blocks = 8192;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_cast, dim3((unsigned)blocks), NTB, 0, s, src, dst, n);
  return hipGetLastError();
}

}  // namespace lsfft_fno
