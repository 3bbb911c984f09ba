// mlp.hip -- training and evaluation kernels of the multiplier surrogate:
// Newton-labelled samples, BF16-MFMA forward and backward with FP32
// gradient accumulation, Adam on FP32 master weights, batched prediction.
#include "kernels.cuh"
#include "mlp.cuh"
#include "mlp_ops.h"

namespace lbm {

using L21 = Lattice<LAT_D2Q21>;

// ---------------------------------------------------------------------------
// master parameter -> BF16 / FP32 operand copies
// ---------------------------------------------------------------------------
// position of input neuron k in a row of the inference copy (the inverse
// of infer_neuron): K block, lane half and slot
__device__ inline int infer_pos(int k) {
  const int q = k >> 5, rem = k & 31, a = rem >> 3, h = (rem >> 2) & 1, s = rem & 3;
  return 16 * (2 * q + (a >> 1)) + 8 * h + 4 * (a & 1) + s;
}

__device__ inline void write_operand(MlpOperands *P, int i, float v) {
  const __bf16 b = (__bf16)v;
  MlpInfer &I = P->inf;
  if (i < MB1) {
    const int n = (i - MW1) / 4, k = (i - MW1) % 4;
    P->w1[n * 16 + k] = b;
    P->w1[n * 16 + 4 + k] = b;
    I.w1[n * 16 + k] = b;
    I.w1[n * 16 + 4 + k] = b;
  } else if (i < MW2) {
    P->b1[i - MB1] = v;
    I.b1[i - MB1] = v;
  } else if (i < MB2) {
    const int n = (i - MW2) / 64, k = (i - MW2) % 64;
    P->w2[n * 64 + k] = b;
    P->w2t[k * 64 + n] = b;
    I.w2[n * 64 + infer_pos(k)] = b;
  } else if (i < MW3) {
    P->b2[i - MB2] = v;
    I.b2[i - MB2] = v;
  } else if (i < MB3) {
    const int n = (i - MW3) / 64, k = (i - MW3) % 64;
    P->w3[n * 64 + k] = b;
    P->w3t[k * 64 + n] = b;
    I.w3[n * 64 + infer_pos(k)] = b;
  } else if (i < MW4) {
    P->b3[i - MB3] = v;
    I.b3[i - MB3] = v;
  } else if (i < MB4) {
    const int n = (i - MW4) / 64, k = (i - MW4) % 64;
    P->w4[n * 64 + k] = b;
    P->w4t[k * 16 + n] = b;
    I.w4hi[n * 64 + infer_pos(k)] = b;
    I.w4lo[n * 64 + infer_pos(k)] = (__bf16)(v - (float)b);
  } else if (i < MMU) {
    P->b4[i - MB4] = v;
    I.b4[i - MB4] = v;
  } else if (i < MSIG) {
    P->mu[i - MMU] = v;
  } else if (i < MLP_NPARAM) {
    P->sig[i - MSIG] = v;
  }
}

__global__ void k_mlp_operands(const float *w, MlpOperands *P) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < MLP_NPARAM) write_operand(P, i, w[i]);
}

// ---------------------------------------------------------------------------
// training set: canonical octant, label statistics, normalised inputs
// ---------------------------------------------------------------------------
// The network learns the canonical octant u_x >= u_y >= 0 (reflection
// symmetry of the lattice): every sample and its label are mapped there in
// place, and each block adds its labels (VAR: squared deviations from mu),
// one partial per block and output, in a fixed order.
template <bool VAR>
__global__ void __launch_bounds__(256) k_mlp_labels(double *x, double *lam, int64_t n, const double *mu,
                                                    double *part) {
  __shared__ double red[4][8];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  double v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = i < n ? lam[i * 8 + k] : 0.0;
  if (!VAR && i < n) {
    double ux = x[i * 4 + 1], uy = x[i * 4 + 2];
    if (ux < 0.0) { ux = -ux; v[1] = -v[1]; v[4] = -v[4]; v[6] = -v[6]; }
    if (uy < 0.0) { uy = -uy; v[2] = -v[2]; v[4] = -v[4]; v[7] = -v[7]; }
    if (uy > ux) {
      double t = ux; ux = uy; uy = t;
      t = v[1]; v[1] = v[2]; v[2] = t;
      t = v[3]; v[3] = v[5]; v[5] = t;
      t = v[6]; v[6] = v[7]; v[7] = t;
    }
    x[i * 4 + 1] = ux;
    x[i * 4 + 2] = uy;
#pragma unroll
    for (int k = 0; k < 8; ++k) lam[i * 8 + k] = v[k];
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    double s = v[k];
    if (VAR) s = i < n ? (s - mu[k]) * (s - mu[k]) : 0.0;
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][k] = s;
  }
  __syncthreads();
  if (threadIdx.x < 8) {
    const int k = threadIdx.x;
    part[(int64_t)blockIdx.x * 8 + k] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
  }
}

// mean (VAR: standard deviation, one where it vanishes) of the labels from
// the partials, one wavefront per output; also into the packed parameters
template <bool VAR>
__global__ void __launch_bounds__(512) k_mlp_label_stats(const double *part, int64_t nblk, int64_t n, double *out,
                                                         float *w) {
  const int k = threadIdx.x >> 6, l = threadIdx.x & 63;
  double s = 0.0;
  for (int64_t b = l; b < nblk; b += 64) s += part[b * 8 + k];
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
  if (l) return;
  s /= (double)n;
  if (VAR) {
    s = sqrt(s);
    if (!(s > 1e-12)) s = 1.0;
  }
  out[k] = s;
  w[(VAR ? MSIG : MMU) + k] = (float)s;
}

__global__ void __launch_bounds__(256) k_mlp_samples(const double *x, const double *lam, int64_t n, const double *mu,
                                                     const double *sg, float *xh, float *th) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  xh[4 * i] = (float)((x[4 * i] - 2.6) / 2.4);
  xh[4 * i + 1] = (float)(x[4 * i + 1] / 2.5);
  xh[4 * i + 2] = (float)(x[4 * i + 2] / 2.5);
  xh[4 * i + 3] = (float)((x[4 * i + 3] - 1.75) / 1.25);
#pragma unroll
  for (int k = 0; k < 8; ++k) th[8 * i + k] = (float)((lam[8 * i + k] - mu[k]) / sg[k]);
}

// ---------------------------------------------------------------------------
// one 32-sample tile per block of four wavefronts: forward, loss, backward.
// A batch is a few dozen blocks, so its time is one block's chain of layers:
// wavefronts 0 and 1 take the two 32-column tiles of the chain (layers, then
// deltas), 2 and 3 the weight gradients that the chain has already passed.
// With one wavefront doing all of it a batch of 1024 took 20.2 us, now 11.5.
// Every tile is the same MFMA sequence whichever wavefront runs it.  Each block
// writes its whole gradient (every trainable entry once) and its loss to a
// slot of its own, gpart[block][MLP_NTRAIN] and lpart[block]; k_mlp_gsum
// adds the slots in block order, so that training is reproducible run to
// run (float atomics would add them in arrival order)
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_mlp_train(const MlpOperands *P, const float *xh, const float *th,
                                                  const int32_t *perm, int64_t off, float inv_count,
                                                  float *gpart, float *lpart) {
  float *grad = gpart + (int64_t)blockIdx.x * MLP_NTRAIN;
  __shared__ __align__(16) __bf16 xin[32 * 16];
  __shared__ __align__(16) __bf16 h1[32 * 64];
  __shared__ __align__(16) __bf16 h2[32 * 64];
  __shared__ __align__(16) __bf16 h3[32 * 64];
  __shared__ __align__(16) __bf16 da[32 * 64];
  __shared__ __align__(16) __bf16 db[32 * 64];
  __shared__ __align__(16) __bf16 dc[32 * 64];
  __shared__ float z[3 * 32 * 64];
  __shared__ float y[32 * 8];
  __shared__ float d4[32 * 8];
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int n0 = 32 * (wv & 1);  // the wavefront's column tile
  const bool chain = wv < 2;
  WTile<64> w3t, w2t;
  if (chain) {
    w3t.load(P->w3t, 64, n0);
    w2t.load(P->w2t, 64, n0);
  }
  const int64_t base = off + (int64_t)blockIdx.x * 32;
  if (threadIdx.x < 32) {
    const int64_t s = perm[base + l];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float x = xh[s * 4 + k];
      const __bf16 hi = (__bf16)x;
      xin[l * 16 + k] = hi;
      xin[l * 16 + 4 + k] = (__bf16)(x - (float)hi);
    }
#pragma unroll
    for (int k = 8; k < 16; ++k) xin[l * 16 + k] = (__bf16)0.0f;
  }
  __syncthreads();
  mlp_forward_tile(P, xin, h1, h2, h3, y, z, wv);
  // Huber loss (delta 0.5) on the normalised outputs and its gradient
  constexpr float HD = 0.5f;
  if (wv == 0) {
    float part = 0.0f;
    if (l < 32) {
      const int64_t s = perm[base + l];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float r = y[l * 8 + k] - th[s * 8 + k];
        const float a = fabsf(r);
        d4[l * 8 + k] = fminf(fmaxf(r, -HD), HD) * inv_count;
        part += a <= HD ? 0.5f * r * r : HD * (a - 0.5f * HD);
      }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) part += __shfl_xor(part, m, 64);
    if (l == 0) lpart[blockIdx.x] = part * inv_count;
  }
  __syncthreads();
  const int kr = 8 * (l >> 5), lc = l & 31;
  // weight gradient tile rows m0.., columns c0.. of a 64 x 64 layer:
  // dW = delta^T h (K = samples)
  auto grad_tile = [&](const __bf16 *dl, const __bf16 *hp, int woff, int m0, int c0) {
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
    for (int k0 = 0; k0 < 32; k0 += 16) {
      bf16x8 a, b;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int s = k0 + kr + j;
        a[j] = dl[s * 64 + m0 + lc];
        b[j] = hp[s * 64 + c0 + lc];
      }
      acc = mfma32(a, b, acc);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) grad[woff + (m0 + c_row(l, r)) * 64 + c0 + lc] = acc[r];
  };
  auto grad_bias = [&](const __bf16 *dl, int boff) {
    float s = 0.0f;
    for (int q = 0; q < 32; ++q) s += (float)dl[q * 64 + l];
    grad[boff + l] = s;
  };
  // delta of the layer below: out = (delta W) .* silu'(z), one column tile
  auto delta_tile = [&](const __bf16 *dl, const WTile<64> &wt, const float *zl, __bf16 *out) {
    const f32x16 acc = gemm_aw<64>(dl, 64, wt);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = c_row(l, r), col = n0 + lc;
      out[row * 64 + col] = (__bf16)(acc[r] * dsilu_f(zl[row * 64 + col]));
    }
  };
  if (chain) {
    // delta3 = (d4 W4) .* silu'(z3)
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    bf16x8 a;
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] = (kr + j) < 8 ? (__bf16)d4[lc * 8 + kr + j] : (__bf16)0.0f;
    const bf16x8 b = *(const bf16x8 *)(P->w4t + (n0 + lc) * 16 + kr);
    acc = mfma32(a, b, acc);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = c_row(l, r), col = n0 + lc;
      da[row * 64 + col] = (__bf16)(acc[r] * dsilu_f(z[4096 + row * 64 + col]));
    }
  } else {
    // dW4 = d4^T h3 (rows: 8 outputs of 32, columns: 64 hidden), K = samples
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
    for (int k0 = 0; k0 < 32; k0 += 16) {
      bf16x8 a, b;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int s = k0 + kr + j;
        a[j] = lc < 8 ? (__bf16)d4[s * 8 + lc] : (__bf16)0.0f;
        b[j] = h3[s * 64 + n0 + lc];
      }
      acc = mfma32(a, b, acc);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = c_row(l, r);
      if (m < 8) grad[MW4 + m * 64 + n0 + lc] = acc[r];
    }
    if (wv == 2 && l < 8) {
      float s = 0.0f;
      for (int q = 0; q < 32; ++q) s += d4[q * 8 + l];
      grad[MB4 + l] = s;
    }
  }
  __syncthreads();
  if (chain) {
    delta_tile(da, w3t, z + 2048, db);
  } else {
    grad_tile(da, h2, MW3, 0, n0);
    grad_tile(da, h2, MW3, 32, n0);
    if (wv == 2) grad_bias(da, MB3);
  }
  __syncthreads();
  if (chain) {
    delta_tile(db, w2t, z, dc);
  } else {
    grad_tile(db, h1, MW2, 0, n0);
    grad_tile(db, h1, MW2, 32, n0);
    if (wv == 2) grad_bias(db, MB2);
  }
  __syncthreads();
  // dW1 = delta1^T xin; the high and low input columns share the weights
  if (chain) {
    const int m0 = n0;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
    for (int k0 = 0; k0 < 32; k0 += 16) {
      bf16x8 a, b;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int s = k0 + kr + j;
        a[j] = dc[s * 64 + m0 + lc];
        b[j] = lc < 16 ? xin[s * 16 + lc] : (__bf16)0.0f;
      }
      acc = mfma32(a, b, acc);
    }
    // columns lc and lc + 4 (the high and low parts of input lc) share
    // the weight: their lanes (same rows) are added before the store
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float v = acc[r] + __shfl_xor(acc[r], 4);
      if (lc < 4) grad[MW1 + (m0 + c_row(l, r)) * 4 + lc] = v;
    }
  } else if (wv == 2) {
    grad_bias(dc, MB1);
  }
}

// Gradient of the batch = the blocks' slots added in block order; the loss is
// accumulated (over the batches of an epoch).  ADAM: and one Adam step
// (Kingma & Ba 2015) on the entry, whose state is read while the slots are,
// so that a batch is two launches.  Sixteen slots are in flight per lane: a
// launch is as long as its rounds of reads (9.9 us one after the other, and
// 4.4 us and a gap for Adam on its own; together 4.8).
template <bool ADAM>
__global__ void __launch_bounds__(64) k_mlp_gsum(const float *gpart, const float *lpart, int nblk, float *grad,
                                                 float *loss, float *w, float *m, float *v, MlpOperands *P, float lr,
                                                 float c1, float c2) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i < MLP_NTRAIN) {
    float wi = 0.0f, mi = 0.0f, vi = 0.0f;
    if (ADAM) {
      wi = w[i];
      mi = m[i];
      vi = v[i];
    }
    float s = 0.0f;
    int b = 0;
    for (; b + 16 <= nblk; b += 16) {
      float p[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) p[q] = gpart[(int64_t)(b + q) * MLP_NTRAIN + i];
#pragma unroll
      for (int q = 0; q < 16; ++q) s += p[q];
    }
    for (; b < nblk; ++b) s += gpart[(int64_t)b * MLP_NTRAIN + i];
    if (ADAM) {
      // (the fused operations spelled out: training amplifies a different
      // rounding, so that the same samples give the same weights only with
      // the same one)
      mi = __builtin_fmaf(s, 0.1f, 0.9f * mi);
      vi = __builtin_fmaf(s, 0.001f * s, 0.999f * vi);
      m[i] = mi;
      v[i] = vi;
      wi = wi - lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
      w[i] = wi;
      write_operand(P, i, wi);
    } else {
      grad[i] = s;
    }
  }
  if (i == MLP_NTRAIN) {  // a lane of the last block
    float s = 0.0f;
    for (int b = 0; b < nblk; ++b) s += lpart[b];
    *loss += s;
  }
}

// ---------------------------------------------------------------------------
// batched prediction of the multipliers from raw states (rho, u_x, u_y, T)
// ---------------------------------------------------------------------------
// (the same inference as the collide: weights staged in LDS once per block,
// one sample per lane)
__global__ void __launch_bounds__(256) k_mlp_predict(const MlpOperands *P, const double *x, int64_t n,
                                                     double *lam) {
  __shared__ MlpInfer W;
  stage_infer(&P->inf, &W);
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool ok = s < n;
  float ux = ok ? (float)x[s * 4 + 1] : 0.0f, uy = ok ? (float)x[s * 4 + 2] : 0.0f;
  const Canon cn = canonical(ux, uy);
  float xin[4], y[8];
  mlp_normalise(ok ? (float)x[s * 4] : 1.0f, ux, uy, ok ? (float)x[s * 4 + 3] : 1.0f, xin);
  mlp_infer_wave(W, xin, y);
  if (ok) {
    double out[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) out[k] = (double)P->mu[k] + (double)P->sig[k] * (double)y[k];
    uncanonical(cn, out);
#pragma unroll
    for (int k = 0; k < 8; ++k) lam[s * 8 + k] = out[k];
  }
}

// ---------------------------------------------------------------------------
// Newton labels: cold start (lambda = 0) per sample; ok = converged
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_mlp_label(const double *x, int64_t n, double tol, int max_it,
                                                   double *lam, uint8_t *ok, int *iters) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  double l8[NLAM], e[L21::Q];
#pragma unroll
  for (int a = 0; a < NLAM; ++a) l8[a] = 0.0;
  const int it = newton_solve<L21>(x[s * 4 + 1], x[s * 4 + 2], x[s * 4 + 3], l8, tol, max_it, e);
  bool good = it >= 0;
#pragma unroll
  for (int a = 0; a < NLAM; ++a) {
    good = good && isfinite(l8[a]);
    lam[s * 8 + a] = l8[a];
  }
  ok[s] = good ? 1 : 0;
  iters[s] = it;
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
void mlp_operands(const float *w, void *P, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_operands, dim3((MLP_NPARAM + 255) / 256), dim3(256), 0, st, w, (MlpOperands *)P);
}

void mlp_prepare(double *x, double *lam, int64_t n, double *part, double *stats, float *w, float *xh, float *th,
                 hipStream_t st) {
  const unsigned nb = (unsigned)((n + 255) / 256);
  double *mu = stats, *sg = stats + 8;
  hipLaunchKernelGGL((k_mlp_labels<false>), dim3(nb), dim3(256), 0, st, x, lam, n, mu, part);
  hipLaunchKernelGGL((k_mlp_label_stats<false>), dim3(1), dim3(512), 0, st, part, (int64_t)nb, n, mu, w);
  hipLaunchKernelGGL((k_mlp_labels<true>), dim3(nb), dim3(256), 0, st, x, lam, n, mu, part);
  hipLaunchKernelGGL((k_mlp_label_stats<true>), dim3(1), dim3(512), 0, st, part, (int64_t)nb, n, sg, w);
  hipLaunchKernelGGL(k_mlp_samples, dim3(nb), dim3(256), 0, st, x, lam, n, mu, sg, xh, th);
}

size_t mlp_prepare_bytes(int64_t n) { return sizeof(double) * (8 * (size_t)((n + 255) / 256) + 16); }

static float *train_tiles(const void *P, const float *xh, const float *th, const int32_t *perm, int64_t off,
                          int64_t count, float *gpart, hipStream_t st) {
  const int nblk = (int)(count / 32);
  float *lpart = gpart + (int64_t)nblk * MLP_NTRAIN;
  hipLaunchKernelGGL(k_mlp_train, dim3((unsigned)nblk), dim3(256), 0, st, (const MlpOperands *)P, xh, th, perm, off,
                     1.0f / (float)(count * 8), gpart, lpart);
  return lpart;
}

void mlp_grad_batch(const void *P, const float *xh, const float *th, const int32_t *perm, int64_t count,
                    float *gpart, float *grad, float *loss, hipStream_t st) {
  const float *lpart = train_tiles(P, xh, th, perm, 0, count, gpart, st);
  hipLaunchKernelGGL((k_mlp_gsum<false>), dim3(MLP_NTRAIN / 64 + 1), dim3(64), 0, st, gpart, lpart,
                     (int)(count / 32), grad, loss, nullptr, nullptr, nullptr, nullptr, 0.0f, 1.0f, 1.0f);
}

void mlp_train_batch(void *P, const float *xh, const float *th, const int32_t *perm, int64_t off, int64_t count,
                     float *gpart, float *loss, float *w, float *m, float *v, float lr, int t, hipStream_t st) {
  const float *lpart = train_tiles(P, xh, th, perm, off, count, gpart, st);
  const float c1 = 1.0f - powf(0.9f, (float)t), c2 = 1.0f - powf(0.999f, (float)t);
  hipLaunchKernelGGL((k_mlp_gsum<true>), dim3(MLP_NTRAIN / 64 + 1), dim3(64), 0, st, gpart, lpart,
                     (int)(count / 32), nullptr, loss, w, m, v, (MlpOperands *)P, lr, c1, c2);
}

size_t mlp_partials_bytes(int64_t count) { return sizeof(float) * (size_t)(count / 32) * (MLP_NTRAIN + 1); }

void mlp_predict(const void *P, const double *x, int64_t n, double *lam, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_predict, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const MlpOperands *)P, x,
                     n, lam);
}

void mlp_label(const double *x, int64_t n, double tol, int max_it, double *lam, uint8_t *ok, int *iters,
               hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_label, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, x, n, tol, max_it, lam,
                     ok, iters);
}

size_t mlp_operands_bytes() { return sizeof(MlpOperands); }

}  // namespace lbm
