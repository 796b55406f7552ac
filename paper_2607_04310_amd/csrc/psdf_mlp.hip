// Screener MLP kernels: inference on feature rows, the training step
// (forward, backward, deterministic gradient reduction, Adam) and the label
// generator (features and exact per-edge pool distances of sampled
// (stage, edge) pairs).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "psdf.h"
#include "psdf_batch.hpp"
#include "psdf_host.hpp"
#include "psdf_mlp.hpp"

namespace psdf {

constexpr int kMlpWaves = 4;          // waves per work-group
constexpr int kGradRow = kMlpParams + 1;   // per-wave partial gradient row (+ loss)

// y[i] for feature rows X[i][0..3], one wave per 16-row group.
__global__ __launch_bounds__(64 * kMlpWaves) void mlp_forward_kernel(const float* __restrict__ th,
                                                                      const float* __restrict__ X,
                                                                      int B, float* __restrict__ y) {
  MlpFrag f;
  mlp_load(th, f);
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int wave = blockIdx.x * kMlpWaves + (threadIdx.x >> 6);
  const int stride = gridDim.x * kMlpWaves;
  for (int grp = wave; grp * 16 < B; grp += stride) {
    const int i = grp * 16 + n;
    float x0 = 0.f, x1 = 0.f, x2 = 0.f, x3 = 0.f;
    if (i < B) { x0 = X[4 * i]; x1 = X[4 * i + 1]; x2 = X[4 * i + 2]; x3 = X[4 * i + 3]; }
    MlpAct a;
    mlp_forward16(f, x0, x1, x2, x3, a);
    if (g == 0 && i < B) y[i] = a.y;
  }
}

// Forward + backward of the mean squared error over B rows.  A work-group
// takes 64 rows at a time (16 per wave), `iters` times, and writes its partial
// gradient (and partial sum of squared errors) to row blockIdx.x of
// part[][kGradRow].
//
// Latency-bound at training sizes (4096 rows: 64 work-groups, one iteration),
// so the passes are arranged to need few dependent steps:
//  * W2 goes to LDS once as BF16, as it is and transposed, so that both its
//    fragments are 8-byte LDS reads (they were 128 gathers per lane);
//  * every layer is taken in two orientations, units x rows and rows x units
//    (the same products with the operands exchanged): a fragment of the
//    second, lane (g, n) = rows 4g .. 4g + 3 of unit n, is at once the
//    operand of the weight gradients, whose contraction runs over rows (they
//    were transposed through LDS element by element), and column sums over
//    rows stay in the lane but for two exchanges (they were four per value);
//  * the waves exchange those fragments through LDS and each accumulates a
//    quarter of dW2 and dW1 over the work-group's 64 rows: one partial row
//    per work-group instead of one per wave.
// Gradient and Adam step of 4096 rows: 15.6 + 11.5 us -> 9.6 + 4.0 us (27.2 ->
// 11.8 us per call, back to back).
constexpr int kW2Stride = kH + 8;   // shorts; rows 16-byte aligned, spread over the banks

__global__ __launch_bounds__(64 * kMlpWaves) void mlp_grad_kernel(const float* __restrict__ th,
                                                                   const float* __restrict__ X,
                                                                   const float* __restrict__ T,
                                                                   int B, int iters,
                                                                   float* __restrict__ part) {
  static_assert(kMlpWaves == 4, "a wave per 16-unit block of the weight gradients");
  __shared__ alignas(16) short w2[kH][kW2Stride], w2t[kH][kW2Stride];
  __shared__ bf16x4 xh1[4][4][64], xdh2[4][4][64], xdh1[4][4][64], xx[4][64];
  __shared__ float colsum[3][4][kH], rowsum[2][4];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, n = lane & 15, g = lane >> 4;

  // W2, four consecutive columns per load
  {
    Float4u v[kH * kH / 4 / 256];
#pragma unroll
    for (int k = 0; k < kH * kH / 4 / 256; ++k)
      v[k] = *reinterpret_cast<const Float4u*>(th + kOffW2 + 4 * (tid + 256 * k));
#pragma unroll
    for (int k = 0; k < kH * kH / 4 / 256; ++k) {
      const int e = 4 * (tid + 256 * k), row = e / kH, col = e % kH;
      bf16x4 q;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        q[r] = to_bf16(v[k].v[r]);
        w2t[col + r][row] = q[r];
      }
      *reinterpret_cast<bf16x4*>(&w2[row][col]) = q;
    }
  }
  // the other parameters, per row of a fragment (o1: unit 16 mb + 4g + r) and
  // per column (o2: unit 16 mb + n)
  bf16x4 a1[4];
  Float4u b1[4], b2[4], w3[4];
  float b1c[4], b2c[4], w3c[4];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) {
    const int u = 16 * mb + n, q = 16 * mb + 4 * g;
    const Float4u f = *reinterpret_cast<const Float4u*>(th + kOffW1 + u * kIn);
#pragma unroll
    for (int r = 0; r < 4; ++r) a1[mb][r] = g == 0 ? to_bf16(f.v[r]) : (short)0;
    b1[mb] = *reinterpret_cast<const Float4u*>(th + kOffB1 + q);
    b2[mb] = *reinterpret_cast<const Float4u*>(th + kOffB2 + q);
    w3[mb] = *reinterpret_cast<const Float4u*>(th + kOffW3 + q);
    b1c[mb] = th[kOffB1 + u];
    b2c[mb] = th[kOffB2 + u];
    w3c[mb] = th[kOffW3 + u];
  }
  const float b3 = th[kOffB3];
  __syncthreads();
  bf16x8 a2[4][2], a2t[4][2];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const int row = 16 * mb + n, c0 = perm_unit(kb, g, 0), c1 = perm_unit(kb, g, 4);
      const bf16x4 p0 = *reinterpret_cast<const bf16x4*>(&w2[row][c0]);
      const bf16x4 p1 = *reinterpret_cast<const bf16x4*>(&w2[row][c1]);
      const bf16x4 t0 = *reinterpret_cast<const bf16x4*>(&w2t[row][c0]);
      const bf16x4 t1 = *reinterpret_cast<const bf16x4*>(&w2t[row][c1]);
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        a2[mb][kb][r] = r < 4 ? p0[r & 3] : p1[r & 3];
        a2t[mb][kb][r] = r < 4 ? t0[r & 3] : t1[r & 3];
      }
    }

  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  f32x4 gW2[4], gW1 = zero4;
  float gb1[4], gb2[4], gw3[4], gb3 = 0.f, sse = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    gW2[q] = zero4;
    gb1[q] = gb2[q] = gw3[q] = 0.f;
  }
  const float inv_b = 2.0f / (float)B;
  for (int it = 0; it < iters; ++it) {
    const long base = ((long)blockIdx.x * iters + it) * 64 + 16 * w;   // the wave's first row
    const long i = base + n;
    Float4u x;
    float t = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) x.v[r] = 0.f;
    if (i < B) {
      x = *reinterpret_cast<const Float4u*>(X + 4 * i);
      t = T[i];
    }
    bf16x4 xt = {0, 0, 0, 0};   // rows x features
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const long row = base + 4 * g + r;
      if (n < kIn && row < B) xt[r] = to_bf16(X[4 * row + n]);
    }
    const bf16x4 none = {0, 0, 0, 0};
    const bf16x4 bx = g == 0 ? mlp_features(x.v[0], x.v[1], x.v[2], x.v[3]) : none;

    // layer 1
    bf16x8 h1[2];    // units x rows: operand of layer 2
    f32x4 e1[4];     // rows x units
    bf16x4 h1c[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1[mb], bx, zero4, 0, 0, 0);
      e1[mb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(bx, a1[mb], zero4, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        h1[mb >> 1][(mb & 1) * 4 + r] = to_bf16(fmaxf(d[r] + b1[mb].v[r], 0.f));
        e1[mb][r] += b1c[mb];
        h1c[mb][r] = to_bf16(fmaxf(e1[mb][r], 0.f));
      }
    }
    // layer 2 and the output
    f32x4 p2[4], e2[4];
    float part_y = 0.f;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      f32x4 d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2[mb][0], h1[0], zero4, 0, 0, 0);
      p2[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a2[mb][1], h1[1], d, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h1[0], a2[mb][0], zero4, 0, 0, 0);
      e2[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h1[1], a2[mb][1], d, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p2[mb][r] += b2[mb].v[r];
        part_y = fmaf(w3[mb].v[r], fmaxf(p2[mb][r], 0.f), part_y);
        e2[mb][r] += b2c[mb];
      }
    }
    part_y += __shfl_xor(part_y, 16);
    part_y += __shfl_xor(part_y, 32);
    const float err = i < B ? part_y + b3 - t : 0.f;
    const float dy = err * inv_b;       // row n
    if (g == 0) { sse += err * err; gb3 += dy; }
    float dyr[4];                       // rows 4g + r
#pragma unroll
    for (int r = 0; r < 4; ++r) dyr[r] = __shfl(dy, 4 * g + r);
    // the output gradient of layer 2, of layer 1
    bf16x8 dh2[2];
    bf16x4 dh2c[4], dh1c[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        dh2[mb >> 1][(mb & 1) * 4 + r] = to_bf16(p2[mb][r] > 0.f ? dy * w3[mb].v[r] : 0.f);
        const float dh = e2[mb][r] > 0.f ? dyr[r] * w3c[mb] : 0.f;
        gw3[mb] = fmaf(dyr[r], fmaxf(e2[mb][r], 0.f), gw3[mb]);
        gb2[mb] += dh;
        dh2c[mb][r] = to_bf16(dh);
      }
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      f32x4 d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dh2[0], a2t[mb][0], zero4, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dh2[1], a2t[mb][1], d, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float dh = e1[mb][r] > 0.f ? d[r] : 0.f;
        gb1[mb] += dh;
        dh1c[mb][r] = to_bf16(dh);
      }
    }
    // the weight gradients: wave w takes units 16 w .. of layer 2 (dW2) and
    // of layer 1 (dW1) over all four waves' rows
    if (it > 0) __syncthreads();   // the previous fragments are read
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      xh1[w][mb][lane] = h1c[mb];
      xdh2[w][mb][lane] = dh2c[mb];
      xdh1[w][mb][lane] = dh1c[mb];
    }
    xx[w][lane] = xt;
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const bf16x4 a = xdh2[v][w][lane];
#pragma unroll
      for (int m1 = 0; m1 < 4; ++m1)
        gW2[m1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, xh1[v][m1][lane], gW2[m1], 0, 0, 0);
      gW1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(xdh1[v][w][lane], xx[v][lane], gW1, 0, 0, 0);
    }
  }
  // ---- the work-group's partial gradient
  float* row = part + (size_t)blockIdx.x * kGradRow;
#pragma unroll
  for (int m1 = 0; m1 < 4; ++m1)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      row[kOffW2 + (16 * w + 4 * g + r) * kH + 16 * m1 + n] = gW2[m1][r];
  if (n < kIn) {
#pragma unroll
    for (int r = 0; r < 4; ++r) row[kOffW1 + (16 * w + 4 * g + r) * kIn + n] = gW1[r];
  }
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) {
    float c[3] = {gb1[mb], gb2[mb], gw3[mb]};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      c[k] += __shfl_xor(c[k], 16);
      c[k] += __shfl_xor(c[k], 32);
      if (g == 0) colsum[k][w][16 * mb + n] = c[k];
    }
  }
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    gb3 += __shfl_xor(gb3, o);
    sse += __shfl_xor(sse, o);
  }
  if (lane == 0) { rowsum[0][w] = gb3; rowsum[1][w] = sse; }
  __syncthreads();
  if (tid < 3 * kH) {
    const int k = tid / kH, u = tid % kH;
    const float c = ((colsum[k][0][u] + colsum[k][1][u]) + colsum[k][2][u]) + colsum[k][3][u];
    row[(k == 0 ? kOffB1 : k == 1 ? kOffB2 : kOffW3) + u] = c;
  } else if (tid < 3 * kH + 2) {
    const int k = tid - 3 * kH;
    row[k == 0 ? kOffB3 : kMlpParams] =
        ((rowsum[k][0] + rowsum[k][1]) + rowsum[k][2]) + rowsum[k][3];
  }
}

// Sum the partial rows into grad[kGradRow]; with lr > 0 also apply one Adam
// step to theta (m, v moments; c1 = 1 - beta1^step, c2 = 1 - beta2^step).
// grad[kMlpParams] receives the mean squared error.  A work-group owns 64
// consecutive columns; wave q adds rows q, q + 4, q + 8, ... in that order
// (eight rows in flight per lane) and wave 0, which has loaded theta and the
// moments meanwhile, adds the four wave sums in wave order, so the result
// does not depend on timing.
constexpr int kReduceWaves = 4;
__global__ __launch_bounds__(64 * kReduceWaves) void mlp_reduce_adam_kernel(
    float* __restrict__ th, float* __restrict__ m, float* __restrict__ v,
    const float* __restrict__ part, int rows, int B, float lr, float c1, float c2,
    float* __restrict__ grad, float* __restrict__ loss) {
  __shared__ float red[kReduceWaves][64];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int p = blockIdx.x * 64 + lane;
  const bool adam = lr > 0.f && p < kMlpParams;
  float t0 = 0.f, m0 = 0.f, v0 = 0.f;
  if (q == 0 && adam) { t0 = th[p]; m0 = m[p]; v0 = v[p]; }
  float s = 0.f;
  if (p < kGradRow) {
    const float* col = part + p;
    constexpr int R = kReduceWaves, U = 8;
    int k = q;
    for (; k + (U - 1) * R < rows; k += U * R) {
      float a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) a[u] = col[(size_t)(k + u * R) * kGradRow];
#pragma unroll
      for (int u = 0; u < U; ++u) s += a[u];
    }
    for (; k < rows; k += R) s += col[(size_t)k * kGradRow];
  }
  red[q][lane] = s;
  __syncthreads();
  if (q != 0 || p >= kGradRow) return;
  s = red[0][lane];
#pragma unroll
  for (int w = 1; w < kReduceWaves; ++w) s += red[w][lane];
  if (p == kMlpParams) {
    if (grad) grad[p] = s / (float)B;
    if (loss) *loss = s / (float)B;
    return;
  }
  if (grad) grad[p] = s;
  if (adam) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float mm = b1 * m0 + (1.f - b1) * s;
    const float vv = b2 * v0 + (1.f - b2) * s * s;
    m[p] = mm;
    v[p] = vv;
    th[p] = t0 - lr * (mm / c1) / (sqrtf(vv / c2) + eps);
  }
}

// Features and labels of sampled (stage, edge) pairs: X[i] = the edge's
// robot-frame endpoints / feature scale; t[i] = the edge's pool distance,
// the minimum over the robot vertices to the edge and over its endpoints to
// the robot edges (Sec. IV-B), clipped to [0, 5] m.
__global__ void screen_label_kernel(const FpConst* __restrict__ fps,
                                    const BatchInst* __restrict__ insts,
                                    const int* __restrict__ stage_inst,
                                    const float* __restrict__ poses, const float* __restrict__ ax,
                                    const float* __restrict__ ay, const float* __restrict__ bx,
                                    const float* __restrict__ by, const int* __restrict__ stage,
                                    const int* __restrict__ edge, int n, int S,
                                    float* __restrict__ X, float* __restrict__ T) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int s = stage[i];
  float f0 = NAN, f1 = NAN, f2 = NAN, f3 = NAN, lab = NAN;
  if (s >= 0 && s < S) {
    const int inst = stage_inst[s];
    const BatchInst in = insts[inst];
    const FpConst& F = fps[inst];
    const int j = edge[i];
    if (j >= 0 && j < in.E) {
      const int ge = in.edge_off + j;
      const float* p = poses + 3 * s;
      float sn, cs;
      sincosf(p[2], &sn, &cs);
      float lax, lay, vx, vy;
      local_point(ax[ge], ay[ge], cs, sn, p[0], p[1], lax, lay);
      local_vector(bx[ge] - ax[ge], by[ge] - ay[ge], cs, sn, vx, vy);
      float iv2, il;
      edge_consts(bx[ge] - ax[ge], by[ge] - ay[ge], F.eps, iv2, il);
      const float lbx = lax + vx, lby = lay + vy;
      float d2 = __builtin_huge_valf();
      for (int l = 0; l < F.m; ++l) {
        float vlx = 0.f, vly = 0.f, elx = 0.f, ely = 0.f, ei = 0.f;
#pragma unroll
        for (int q = 0; q < kMaxFp; ++q)
          if (q == l) { vlx = F.vx[q]; vly = F.vy[q]; elx = F.ex[q]; ely = F.ey[q]; ei = F.einv[q]; }
        d2 = fminf(d2, seg_d2(vlx, vly, lax, lay, vx, vy, iv2));
        d2 = fminf(d2, seg_d2(lax, lay, vlx, vly, elx, ely, ei));
        d2 = fminf(d2, seg_d2(lbx, lby, vlx, vly, elx, ely, ei));
      }
      const float sc = 1.0f / kFeatureScale;
      f0 = lax * sc; f1 = lay * sc; f2 = lbx * sc; f3 = lby * sc;
      lab = fminf(fmaxf(sqrtf(d2), 0.f), 5.0f);
    }
  }
  X[4 * i] = f0; X[4 * i + 1] = f1; X[4 * i + 2] = f2; X[4 * i + 3] = f3;
  T[i] = lab;
}

hipError_t launch_labels(const FpConst* fps, const BatchInst* insts, const int* stage_inst,
                         const float* poses, const float* ax, const float* ay, const float* bx,
                         const float* by, const int* stage, const int* edge, int n, int S, float* X,
                         float* T, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  screen_label_kernel<<<(n + 255) / 256, 256, 0, st>>>(fps, insts, stage_inst, poses, ax, ay, bx,
                                                        by, stage, edge, n, S, X, T);
  return hipGetLastError();
}

// Partial rows of B rows of data (one per work-group: 64 rows at a time, at
// most one work-group per CU), and the rows the workspace holds.
constexpr int kGradRowsMax = 256;
static int grad_blocks(int B) {
  return std::min(kGradRowsMax, std::max(1, (B - 1) / 64 + 1));
}
static int grad_ws_rows(int B) {
  return std::min(kGradRowsMax, ((B - 1) / 16 + kMlpWaves) / kMlpWaves * kMlpWaves);
}

}  // namespace psdf

using namespace psdf;

extern "C" {

int psdf_mlp_forward(const float* theta, const float* X, int32_t B, float* y, hipStream_t stream) {
  clear_error();
  if (B < 0) return set_error(PSDF_EINVAL, "B = %d", B);
  if (B == 0) return PSDF_OK;
  if (!theta || !X || !y) return set_error(PSDF_EINVAL, "NULL argument");
  const int groups = (B + 15) / 16;
  const int blocks = (groups + kMlpWaves - 1) / kMlpWaves;
  mlp_forward_kernel<<<blocks < 4096 ? blocks : 4096, 64 * kMlpWaves, 0, stream>>>(theta, X, B, y);
  return hip_status(hipGetLastError());
}

size_t psdf_mlp_ws_bytes(int32_t B) {
  if (B <= 0) return 0;
  return (size_t)grad_ws_rows(B) * kGradRow * sizeof(float);
}

static int mlp_step(float* theta, float* m, float* v, int32_t step, float lr, const float* X,
                    const float* T, int32_t B, float* grad, float* loss, void* ws, size_t ws_bytes,
                    hipStream_t stream) {
  if (B <= 0) return set_error(PSDF_EINVAL, "B = %d", B);
  if (!theta || !X || !T) return set_error(PSDF_EINVAL, "NULL argument");
  if (!ws || ws_bytes < psdf_mlp_ws_bytes(B))
    return set_error(PSDF_EWS, "workspace of %zu bytes, %zu needed", ws_bytes, psdf_mlp_ws_bytes(B));
  const int blocks = grad_blocks(B);
  const int iters = ((B - 1) / 64 + blocks) / blocks;
  float* part = static_cast<float*>(ws);
  mlp_grad_kernel<<<blocks, 64 * kMlpWaves, 0, stream>>>(theta, X, T, B, iters, part);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return hip_status(err);
  const float c1 = (float)(1.0 - std::pow((double)0.9f, step));
  const float c2 = (float)(1.0 - std::pow((double)0.999f, step));
  mlp_reduce_adam_kernel<<<(kGradRow + 63) / 64, 64 * kReduceWaves, 0, stream>>>(
      theta, m, v, part, blocks, B, lr, c1, c2, grad, loss);
  return hip_status(hipGetLastError());
}

int psdf_mlp_grad(const float* theta, const float* X, const float* T, int32_t B, float* grad,
                  void* ws, size_t ws_bytes, hipStream_t stream) {
  clear_error();
  if (!grad) return set_error(PSDF_EINVAL, "grad is NULL");
  return mlp_step(const_cast<float*>(theta), nullptr, nullptr, 1, 0.f, X, T, B, grad, nullptr, ws,
                  ws_bytes, stream);
}

int psdf_mlp_train_step(float* theta, float* m, float* v, int32_t step, float lr, const float* X,
                        const float* T, int32_t B, float* loss, void* ws, size_t ws_bytes,
                        hipStream_t stream) {
  clear_error();
  if (!m || !v || step < 1 || !(lr > 0.f)) return set_error(PSDF_EINVAL, "bad Adam state");
  return mlp_step(theta, m, v, step, lr, X, T, B, nullptr, loss, ws, ws_bytes, stream);
}

}  // extern "C"
