// Host-side launch interface of the surrogate kernels (fno_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>

#include <cstdint>

namespace lsfft_fno {

constexpr int kWidth = 32;   // channels of the hidden layers (one MFMA tile)

// Pointwise layer of kWidth output channels, out[b][o][v] = sum_i w[o][i]
// in[b][i][v] (+ bias[o]) (+ add[b][o][v]); then, if aux, out *=
// GELU'(aux[b][o][v]); if out_act, out_act = GELU(out).  out may be null when
// only out_act is wanted.  w is bf16 [opad][ipad], zero padded, opad kWidth and ipad
// 16 or 32; add needs ipad 32, aux needs add.
struct PwArgs {
  const float* in;
  const __hip_bfloat16* w;
  const float* bias;
  const float* add;
  const float* aux;
  float* out;
  float* out_act;
  int I, ipad, O, opad, B;
  long long V;
};
hipError_t launch_pointwise(const PwArgs& a, hipStream_t s);

// Weight gradient of a pointwise layer of at most 32 channels each way: per block
// partial sums part[blk][32][32] and, after them, [32] of sum_{b,v} g[b][o][v]
// h[b][i][v] and sum g[b][o][v]; then the fixed-order reduction into the packed
// gradient gw [O][I], gb [O].
struct WgArgs {
  const float* g;
  const float* h;
  float* part;
  int O, I, B;
  long long V;
  int nblk;
};
hipError_t launch_wgrad(const WgArgs& a, float* gw, float* gb, hipStream_t s);
int wgrad_blocks(int B, long long V);

// Projection y = W2 gelu(W1 h + b1) + b2 of h [B][32][V]: w1 bf16
// [hidden][32], w2 bf16 [32][hidden] (rows beyond O zero).
struct ProjArgs {
  const float* h;
  const __hip_bfloat16 *w1, *w2;
  const float *b1, *b2;
  float* y;
  int hidden, O, B;
  long long V;
};
hipError_t launch_project(const ProjArgs& a, hipStream_t s);

// Its backward pass: out [B][32][V] = (W1^T dz) gelu'(pre), dz = (W2^T dy)
// gelu'(W1 h + b1), and the packed gradients of both layers.  w1t bf16
// [32][hidden], w2t bf16 [hidden][opad16]; part1, part2: partial sums of
// project_bwd_blocks workgroups, hidden 32 + hidden and 32 hidden + 32 floats
// each.  hidden 32, 64, 128 or 256 (hipErrorInvalidValue otherwise).
struct ProjBwdArgs {
  const float *h, *dy, *pre;
  const __hip_bfloat16 *w1, *w1t, *w2t;
  const float* b1;
  float *out, *part1, *part2;
  int hidden, O, opad16, B;
  long long V;
};
int project_bwd_blocks(int B, long long V, int hidden);
hipError_t launch_project_bwd(const ProjBwdArgs& a, float* gw1, float* gb1, float* gw2, float* gb2, hipStream_t s);

// The kept modes of a batch are laid out in groups of eight,
// md[m / 8][bc][m % 8] (bc = 32 sample + channel); mode_slots(nmodes) modes of
// storage per bc.
inline long long mode_slots(long long nmodes) { return (nmodes + 7) / 8 * 8; }

// Per-mode complex products on bf16 MFMA (x, g and mode 0 / 1's out as md):
//  mode 0: out[m][b][o] = sum_i x[m][b][i] r[m][i][o]
//  mode 1: out[m][b][i] = sum_o x[m][b][o] conj(r[m][i][o])
//  mode 2: out[m][i][o] (fp32 re,im, mode after mode) = sum_b conj(x[m][b][i]) g[m][b][o]
hipError_t launch_modemix(int mode, const float2* x, const __hip_bfloat16* r, const float2* g, float* out,
                          int nmodes, int B, hipStream_t s);

// Truncated transforms over [BC][n][n][n] (x fastest), kept modes as above.
//  forward: md = scale(kx) * sum_x h e^{-i k.x}, scale = sc0 (kx = 0) or sc1
//  inverse: out[bc][x] = sum_kept c(kx) Re(md e^{+i k.x}), c = c0 or c1
hipError_t launch_dft_forward(int n, int M, int BC, const float* h, float2* md, float sc0, float sc1,
                              const float2* tw, hipStream_t s);
hipError_t launch_dft_inverse(int n, int M, int BC, const float2* md, float* out, float c0, float c1,
                              const float2* tw, hipStream_t s);

// loss = mean_b ||y_b - t_b|| / ||t_b||, dy = (y - t) / (||y_b - t_b|| ||t_b|| B)
hipError_t launch_loss(const float* y, const float* t, float* dy, int B, long long per_sample, double* part,
                       int nchunk, double* loss_dev, hipStream_t s);

hipError_t launch_adam(float* p, const float* g, float* m, float* v, long long n, float lr, float b1, float b2,
                       float eps, float bc1, float bc2, hipStream_t s);

// dst[r][c] (bf16, drows x dcols) = src[r * sr + c * sc] inside rows x cols, else 0
hipError_t launch_cast_pad(const float* src, int rows, int cols, long long sr, long long sc, __hip_bfloat16* dst,
                           int drows, int dcols, hipStream_t s);
hipError_t launch_cast(const float* src, __hip_bfloat16* dst, long long n, hipStream_t s);

}  // namespace lsfft_fno
