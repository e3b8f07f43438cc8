// Supervised training of the fused-op estimator (Sec. 3.3.3) on gfx950, fp32.
//
// One pass = forward with the activations of every layer kept, the loss of Eq. (1) read as the
// mean squared difference of logarithms, and the reverse pass of exactly the forward formulas:
//     y = z2.w3 + b3,  z2 = ReLU(z1 W2 + b2),  z1 = ReLU(r W1 + b1),  r = sum of h_L over the
//     ops of the fused op (Secs. 3.3.1, 3.3.2),
//     h_{l+1} = ReLU([h_l | mean over predecessors | mean over successors] W_l + b_l).
// Dense products: forward on the fp32 matrix cores (32x32x2) through the layer update kernel; the reverse pass
// on the bf16 ones in three pieces (dense32.hip): data gradients, and weight gradients, whose contraction
// index is the row of the batch (transposed-A product, split over slabs of rows, partial
// results reduced in a fixed order, so a pass is bit-reproducible).  Everything else is
// bandwidth-bound and done by plain grid-stride kernels.  Adam as published by Kingma & Ba.
#include "common.h"

namespace dc {
namespace {

// ---- sample of each row: largest g with node_off[g] <= v (graphs may be empty) ----
__global__ __launch_bounds__(256) void gid_kernel(const int* __restrict__ node_off, int B, int* __restrict__ gid,
                                                  const int* __restrict__ status) {
  if (status[0] != 0) return;
  const long long ntot = node_off[B];
  for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < ntot;
       v += (long long)gridDim.x * blockDim.x) {
    int lo = 0, hi = B;                 // invariant: node_off[lo] <= v < node_off[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (node_off[mid] <= v) lo = mid; else hi = mid;
    }
    gid[v] = lo;
  }
}

// ---- r[g] = sum over the rows of graph g, fp64 in ascending row order ----
__global__ __launch_bounds__(256) void readout_kernel(const float* __restrict__ h, int H,
                                                      const int* __restrict__ node_off, int B,
                                                      float* __restrict__ R, const int* __restrict__ status) {
  if (status[0] != 0) return;
  const int cpr = H / 4;
  const long long total = (long long)B * cpr;
  const float4* __restrict__ h4 = reinterpret_cast<const float4*>(h);
  for (long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (long long)gridDim.x * blockDim.x) {
    const int g = (int)(idx / cpr), ch = (int)(idx - (long long)g * cpr);
    double a0 = 0, a1 = 0, a2 = 0, a3 = 0;
    const int v1 = node_off[g + 1];
    int v = node_off[g];
    // eight rows requested together, added one after another: the chain of a long sample is eight times shorter
    // (1.8 k rows in 130 samples: 27 -> 8 us)
    for (; v + 8 <= v1; v += 8) {
      float4 x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = h4[(size_t)(v + u) * cpr + ch];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        a0 += x[u].x; a1 += x[u].y; a2 += x[u].z; a3 += x[u].w;
      }
    }
    for (; v < v1; ++v) {
      const float4 x = h4[(size_t)v * cpr + ch];
      a0 += x.x; a1 += x.y; a2 += x.z; a3 += x.w;
    }
    reinterpret_cast<float4*>(R)[idx] = make_float4((float)a0, (float)a1, (float)a2, (float)a3);
  }
}

// ---- per sample: y, the loss term and dL/dy; one wave per sample ----
__global__ __launch_bounds__(256) void loss_kernel(const float* __restrict__ Z2, int H, const float* __restrict__ w3b3,
                                                   const float* __restrict__ target, int B, float floor_,
                                                   float* __restrict__ y, float* __restrict__ dy,
                                                   double* __restrict__ lterm, float* __restrict__ pred,
                                                   int* __restrict__ status) {
  if (status[0] != 0) return;
  const int lane = threadIdx.x & 63;
  const int wpb = blockDim.x >> 6;
  for (int g = blockIdx.x * wpb + (threadIdx.x >> 6); g < B; g += gridDim.x * wpb) {
    // a profiled time is positive and finite: anything else has no logarithm, and the call is refused
    // (every later kernel of the call sees the status word and leaves its outputs alone)
    const float tg = target[g];
    if (!(tg > 0.f) || tg > 3.0e38f) {
      if (lane == 0) set_error(status, DC_ERR_INVALID_ARG);
      continue;
    }
    double s = 0.0;
    for (int j = lane; j < H; j += 64) s += (double)Z2[(size_t)g * H + j] * (double)w3b3[j];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) {
      const float yf = (float)(s + (double)w3b3[H]);
      const double yc = yf > floor_ ? (double)yf : (double)floor_;
      const double dl = log(yc) - log((double)tg);
      y[g] = yf;
      if (pred) pred[g] = yf;
      lterm[g] = dl * dl;
      dy[g] = yf > floor_ ? (float)(2.0 / (double)B * dl / yc) : 0.f;
    }
  }
}

// ---- loss = mean of the terms; one workgroup, fixed order ----
__global__ __launch_bounds__(1024) void loss_reduce_kernel(const double* __restrict__ lterm, int B,
                                                           float* __restrict__ loss,
                                                           const int* __restrict__ status) {
  if (status[0] != 0) return;
  __shared__ double red[1024];
  double s = 0.0;
  for (int g = threadIdx.x; g < B; g += 1024) s += lterm[g];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[0] = B > 0 ? (float)(red[0] / (double)B) : 0.f;
}

// ---- dz2[g][j] = dy[g] w3[j] where z2 > 0 ----
__global__ __launch_bounds__(256) void dz2_kernel(const float* __restrict__ Z2, const float* __restrict__ dy,
                                                  const float* __restrict__ w3, int H, int B,
                                                  float* __restrict__ dZ2, const int* __restrict__ status) {
  if (status[0] != 0) return;
  const long long total = (long long)B * H;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int g = (int)(i / H), j = (int)(i - (long long)g * H);
    dZ2[i] = Z2[i] > 0.f ? dy[g] * w3[j] : 0.f;
  }
}

// ---- x = 0 where the activation is not positive (ReLU'), rows from a device count ----
__global__ __launch_bounds__(256) void relu_mask_kernel(float* __restrict__ x, const float* __restrict__ act,
                                                        const int* __restrict__ nrows, int H,
                                                        const int* __restrict__ status) {
  if (status[0] != 0) return;
  const long long total = (long long)nrows[0] * H;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x)
    if (!(act[i] > 0.f)) x[i] = 0.f;
}

// ---- gradient at the last layer's pre-activations: every op of a fused op receives dr ----
__global__ __launch_bounds__(256) void top_kernel(const float* __restrict__ dR, const int* __restrict__ gid,
                                                  const float* __restrict__ hL, const int* __restrict__ nrows, int H,
                                                  float* __restrict__ dZ, const int* __restrict__ status) {
  if (status[0] != 0) return;
  const int cpr = H / 4;
  const long long total = (long long)nrows[0] * cpr;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const long long v = i / cpr;
    const int ch = (int)(i - v * cpr);
    const float4 g = reinterpret_cast<const float4*>(dR)[(size_t)gid[v] * cpr + ch];
    const float4 a = reinterpret_cast<const float4*>(hL)[i];
    reinterpret_cast<float4*>(dZ)[i] = make_float4(a.x > 0.f ? g.x : 0.f, a.y > 0.f ? g.y : 0.f,
                                                   a.z > 0.f ? g.z : 0.f, a.w > 0.f ? g.w : 0.f);
  }
}

// ---- reverse of the two neighbour means, plus the node's own block, then ReLU' of the layer below ----
// dA [rows, 3d] = dZ W^T holds per row v the gradient at [h[v] | mean over pred(v) | mean over succ(v)].
// h[u] enters the predecessor mean of each successor v with weight 1/indeg(v), and the successor
// mean of each predecessor v with weight 1/outdeg(v).
__global__ __launch_bounds__(256) void gather_back_kernel(const float* __restrict__ dA, int d,
                                                          const int* __restrict__ in_rp, const int* __restrict__ in_ci,
                                                          const int* __restrict__ out_rp,
                                                          const int* __restrict__ out_ci,
                                                          const float* __restrict__ h, const int* __restrict__ nrows,
                                                          float* __restrict__ dZ, const int* __restrict__ status) {
  if (status[0] != 0) return;
  const int cpr = d / 4;
  const long long total = (long long)nrows[0] * cpr;
  const float4* __restrict__ A4 = reinterpret_cast<const float4*>(dA);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const long long u = i / cpr;
    const int ch = (int)(i - u * cpr);
    float4 acc = A4[(size_t)u * 3 * cpr + ch];
    for (int k = out_rp[u]; k < out_rp[u + 1]; ++k) {
      const int v = out_ci[k];
      const float sc = 1.0f / (float)(in_rp[v + 1] - in_rp[v]);
      const float4 x = A4[(size_t)v * 3 * cpr + cpr + ch];
      acc.x += x.x * sc; acc.y += x.y * sc; acc.z += x.z * sc; acc.w += x.w * sc;
    }
    for (int k = in_rp[u]; k < in_rp[u + 1]; ++k) {
      const int v = in_ci[k];
      const float sc = 1.0f / (float)(out_rp[v + 1] - out_rp[v]);
      const float4 x = A4[(size_t)v * 3 * cpr + 2 * cpr + ch];
      acc.x += x.x * sc; acc.y += x.y * sc; acc.z += x.z * sc; acc.w += x.w * sc;
    }
    const float4 a = reinterpret_cast<const float4*>(h)[i];
    reinterpret_cast<float4*>(dZ)[i] = make_float4(a.x > 0.f ? acc.x : 0.f, a.y > 0.f ? acc.y : 0.f,
                                                   a.z > 0.f ? acc.z : 0.f, a.w > 0.f ? acc.w : 0.f);
  }
}

// ---- gradient of the last layer's weights: sum over rows r of A[r][:] y[r], and the sum of y, per slab of rows ----
__global__ __launch_bounds__(512) void wgrad_vector_kernel(const float* __restrict__ A, int d, const float* __restrict__ y,
                                                           const int* __restrict__ nrows, float* __restrict__ part,
                                                           long long part_stride, int S, const int* __restrict__ status) {
  if (status[0] != 0) return;
  const int rows = nrows[0], per = (rows + S - 1) / S;
  const int r0 = min(blockIdx.x * per, rows), r1 = min(r0 + per, rows);
  float* P = part + (size_t)blockIdx.x * (size_t)part_stride;
  for (int j = threadIdx.x; j <= d; j += blockDim.x) {
    float s = 0.f;
    int r = r0;
    if (j < d) {
      for (; r + 8 <= r1; r += 8) {                    // eight rows requested together
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = A[(size_t)(r + u) * d + j];
#pragma unroll
        for (int u = 0; u < 8; ++u) s = fmaf(x[u], y[r + u], s);
      }
      for (; r < r1; ++r) s = fmaf(A[(size_t)r * d + j], y[r], s);
    } else {
      for (; r < r1; ++r) s += y[r];
    }
    P[j] = s;
  }
}

// gW [M*N] and gb [N] = sums of the slabs' partial results, fp64, ascending slab order.  Bound by memory latency: a
// thread owns one sum, so sixteen of its addends are requested together (one at a time, a round trip per slab, took
// 33 us for 128 slabs of 49 k entries; 5.6 us now).  S is a multiple of eight.
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(const float* __restrict__ part, long long part_stride,
                                                           int S, long long MN, int N, float* __restrict__ gW,
                                                           float* __restrict__ gb, const int* __restrict__ status) {
  if (status[0] != 0) return;
  const long long total = MN + (gb ? N : 0);
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    double s = 0.0;
    const float* __restrict__ p = part + i;
    int k = 0;
    for (; k + 16 <= S; k += 16, p += 16 * part_stride) {
      float x[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) x[u] = p[u * part_stride];
#pragma unroll
      for (int u = 0; u < 16; ++u) s += (double)x[u];
    }
    for (; k < S; ++k, p += part_stride) s += (double)*p;
    if (i < MN) gW[i] = (float)s; else gb[i - MN] = (float)s;
  }
}

__global__ void set_count_kernel(int* cnt, int n) {
  cnt[0] = 0;
  cnt[1] = n;
}

__global__ __launch_bounds__(256) void adam_kernel(float* __restrict__ theta, const float* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v, long long n,
                                                   float lr, float beta1, float beta2, float eps, float c1, float c2,
                                                   const int* __restrict__ status) {
  if (status[0] != 0) return;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long long)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = beta1 * m[i] + (1.f - beta1) * gi;
    const float vi = beta2 * v[i] + (1.f - beta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    theta[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);      // c1 = 1/(1-beta1^t), c2 = 1/(1-beta2^t)
  }
}

int grid_for(long long items, int n_cu) {
  long long g = (items + 255) / 256;
  const long long cap = (long long)n_cu * 16;
  if (g > cap) g = cap;
  return g < 1 ? 1 : (int)g;
}

// slabs of a product with ntile tiles: one round of workgroups at two per CU, a multiple of 8
int slabs_for(int ntile, int n_cu, int cap) {
  int S = ((2 * n_cu) / ntile) & ~7;
  if (S > cap) S = cap;
  return S < 8 ? 8 : S;
}

void reduce_slabs(const TrainPass& t, int S, int MN, int N, float* gW, float* gb, hipStream_t s) {
  const long long stride = (long long)MN + N;
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3(grid_for(stride, t.n_cu)), dim3(256), 0, s, t.part, stride, S, (long long)MN, N,
                     gW, gb, t.status);
}

// C = sum over rows of [A0|A1|A2]^T B into gW (and column sums of B into gb)
void weight_gradient(const TrainPass& t, const float* A0, const float* A1, const float* A2, int d, int nseg,
                     const float* Bm, int N, const int* nrows, float* gW, float* gb, hipStream_t s) {
  const int M = nseg * d;
  const int S = slabs_for(wgrad_split_tiles(M, N), t.n_cu, t.slabs);
  launch_wgrad_split(A0, A1, A2, d, nseg, Bm, N, N, nrows, t.part, (long long)M * N + N, S, t.status, s);
  reduce_slabs(t, S, M * N, N, gW, gb, s);
}

// out = dZ W^T for W [N, K] with N = g.H, K = H; WTs: its place in TrainPass::WTs
void data_gradient(const GnnArgs& g, const float* dZ, int H, const float* W, const unsigned short* WTs, float* out, hipStream_t s) {
  if (H >= kSplitLeastReverse) launch_update_split(g, dZ, nullptr, nullptr, H, 1, W, WTs, nullptr, out, s, true);
  else launch_dense_update(g, dZ, nullptr, nullptr, H, 1, WTs, nullptr, out, s);
}

}  // namespace

int train_slabs(int n_cu, int F, int H) {
  // the largest slab count weight_gradient() uses (the partial-result buffer is sized for it)
  (void)n_cu;
  (void)F;
  (void)H;
  return 128;
}

hipError_t launch_train_pass(const TrainPass& t, Profiler* prof, hipStream_t s) {
  auto begin = [&](int fam) { if (prof) prof->begin(fam, s); };
  auto end = [&]() { if (prof) prof->end(s); };
  const int B = t.n_samples, H = t.H, F = t.F, L = t.L;
  const size_t HH = (size_t)H * H;
  const int* nrows = t.node_off + B;          // device-resident row count
  GnnArgs g{};
  g.n_cand = B;
  g.node_off = t.node_off;
  g.out_rowptr = t.out_rowptr;
  g.out_col = t.out_col;
  g.in_rowptr = t.in_rowptr;
  g.in_col = t.in_col;
  g.H = H;
  g.bf16 = 0;
  g.status = t.status;
  g.n_cu = t.n_cu;
  GnnArgs gh = g;                              // the regression network: one row per sample
  gh.n_cand = 1;
  gh.node_off = t.cnt;
  const long long rows_cap = t.max_rows;
  const size_t dmax = (size_t)(F > H ? F : H);
  const float* W1 = t.head;
  const float* b1 = W1 + HH;
  const float* W2 = b1 + H;
  const float* b2 = W2 + HH;
  const float* w3 = b2 + H;                    // followed by b3
  // gradient vector: W_layers | b_layers | W1 b1 W2 b2 w3 b3
  size_t nW = 0;
  for (int l = 0; l < L; ++l) nW += (size_t)3 * (l == 0 ? F : H) * H;
  float* gWl = t.grad;
  float* gbl = t.grad + nW;
  float* gW1 = gbl + (size_t)L * H;
  float* gb1 = gW1 + HH;
  float* gW2 = gb1 + H;
  float* gb2 = gW2 + HH;
  float* gw3 = gb2 + H;
  float* gb3 = gw3 + H;

  hipLaunchKernelGGL(set_count_kernel, dim3(1), dim3(1), 0, s, t.cnt, B);
  hipLaunchKernelGGL(gid_kernel, dim3(grid_for(rows_cap, t.n_cu)), dim3(256), 0, s, t.node_off, B, t.gid, t.status);

  // ---- forward, every layer's output kept ----
  // In fp32 instructions: a sum that rounds differently about zero passes or stops a row's whole gradient at its ReLU, and in
  // 475 k rows some do (gradients of either form 4e-6 to 9e-6 apart, each as far from 64 bits; the reverse pass alone: 1.4e-7).
  const float* hcur = t.X;
  int d = F;
  const float* Wl = t.W;
  const float* bl = t.b;
  for (int l = 0; l < L; ++l) {
    float* hn = t.hs + (size_t)l * rows_cap * H;
    float* mp = t.means + (size_t)(2 * l) * rows_cap * dmax;      // both means are kept for the reverse pass
    float* ms = mp + (size_t)rows_cap * dmax;
    begin(kFamTrainAggregate);
    launch_mean_aggregate(g, hcur, d, mp, ms, s);
    end();
    begin(kFamTrainUpdate);
    launch_dense_update(g, hcur, mp, ms, d, 3, Wl, bl, hn, s);
    end();
    Wl += (size_t)3 * d * H;
    bl += H;
    hcur = hn;
    d = H;
  }
  begin(kFamTrainHead);
  hipLaunchKernelGGL(readout_kernel, dim3(grid_for((long long)B * (H / 4), t.n_cu)), dim3(256), 0, s, hcur, H,
                     t.node_off, B, t.R, t.status);
  launch_dense_update(gh, t.R, nullptr, nullptr, H, 1, W1, b1, t.Z1, s);
  launch_dense_update(gh, t.Z1, nullptr, nullptr, H, 1, W2, b2, t.Z2, s);
  hipLaunchKernelGGL(loss_kernel, dim3(grid_for((long long)B * 64, t.n_cu)), dim3(256), 0, s, t.Z2, H, w3, t.target, B,
                     t.floor, t.y, t.dy, t.lterm, t.pred, t.status);
  hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(1024), 0, s, t.lterm, B, t.loss, t.status);
  if (!t.grad) {
    end();
    return hipGetLastError();
  }

  // ---- regression network, reverse ----
  const unsigned short* WTs = t.WTs + (size_t)(L - 1) * 9 * HH;
  const int* nB = t.cnt + 1;
  hipLaunchKernelGGL(wgrad_vector_kernel, dim3(t.slabs), dim3(512), 0, s, t.Z2, H, t.dy, nB, t.part, (long long)H + 1, t.slabs, t.status);
  reduce_slabs(t, t.slabs, H, 1, gw3, gb3, s);
  hipLaunchKernelGGL(dz2_kernel, dim3(grid_for((long long)B * H, t.n_cu)), dim3(256), 0, s, t.Z2, t.dy, w3, H, B,
                     t.dZ2, t.status);
  weight_gradient(t, t.Z1, nullptr, nullptr, H, 1, t.dZ2, H, nB, gW2, gb2, s);
  data_gradient(gh, t.dZ2, H, W2, WTs + 3 * HH, t.dZ1, s);
  hipLaunchKernelGGL(relu_mask_kernel, dim3(grid_for((long long)B * H, t.n_cu)), dim3(256), 0, s, t.dZ1, t.Z1, nB, H,
                     t.status);
  weight_gradient(t, t.R, nullptr, nullptr, H, 1, t.dZ1, H, nB, gW1, gb1, s);
  data_gradient(gh, t.dZ1, H, W1, WTs, t.dR, s);

  // ---- graph layers, reverse ----
  float* dZ = t.dZ[0];
  float* dZn = t.dZ[1];
  hipLaunchKernelGGL(top_kernel, dim3(grid_for(rows_cap * (H / 4), t.n_cu)), dim3(256), 0, s, t.dR, t.gid, hcur, nrows,
                     H, dZ, t.status);
  end();
  GnnArgs g3 = g;
  g3.H = 3 * H;                                // dA = dZ W^T is [rows, 3H] for the layers above the first
  for (int l = L - 1; l >= 0; --l) {
    const int dl = l == 0 ? F : H;
    const float* hl = l == 0 ? t.X : t.hs + (size_t)(l - 1) * rows_cap * H;
    size_t woff = 0;
    for (int k = 0; k < l; ++k) woff += (size_t)3 * (k == 0 ? F : H) * H;
    const float* mp = t.means + (size_t)(2 * l) * rows_cap * dmax;
    const float* ms = mp + (size_t)rows_cap * dmax;
    begin(kFamTrainWgrad);
    weight_gradient(t, hl, mp, ms, dl, 3, dZ, H, nrows, gWl + woff, gbl + (size_t)l * H, s);
    end();
    if (l == 0) break;
    begin(kFamTrainDgrad);
    data_gradient(g3, dZ, H, t.W + woff, t.WTs + (size_t)(l - 1) * 9 * HH, t.dA, s);
    end();
    begin(kFamTrainGatherBack);
    hipLaunchKernelGGL(gather_back_kernel, dim3(grid_for(rows_cap * (H / 4), t.n_cu)), dim3(256), 0, s, t.dA, H,
                       t.in_rowptr, t.in_col, t.out_rowptr, t.out_col, hl, nrows, dZn, t.status);
    end();
    float* tmp = dZ;
    dZ = dZn;
    dZn = tmp;
  }
  return hipGetLastError();
}

hipError_t launch_adam(float* theta, const float* grad, float* m, float* v, long long n, float lr, float beta1,
                       float beta2, float eps, double c1, double c2, const int* status, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(adam_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, theta, grad, m, v, n, lr, beta1, beta2,
                     eps, (float)c1, (float)c2, status);
  return hipGetLastError();
}

}  // namespace dc
