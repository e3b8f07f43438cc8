// Neighbourhood encoding with attention coefficients (Sec. 3.3.1, first equation; gfx950).
//
// The paper gives K heads, one weight matrix per head and a coefficient gamma^k_ij per
// neighbour j of node i (i included) without a formula for gamma; this build takes it as
// graph attention networks do:
//     z_j = W e'_j,   u_ij = LeakyReLU_0.2(a_src . z_i + a_dst . z_j)   per head,
//     gamma_ij = softmax over j in N_i,   e_i = ReLU(sum_j gamma_ij z_j + b),
// with N_i = (i, predecessors ascending, successors ascending) and heads being contiguous
// blocks of H / K columns.  z = h W is a dense contraction (update_kernel); here are the
// two kernels that follow it: the score terms per node and head (with H = 256, bf16 and up to four heads the product
// forms them itself, gnn_layer256.hip), and the weighted sums.
//
// A row of z is served by LPR = H / 8 lanes, eight columns each (16 bytes in bf16, 32 in
// fp32); a head's Dh = H / K columns sit in Dh / 8 adjacent lanes, so the reductions over a
// head are butterflies over those lanes.  H and K are powers of two, Dh >= 8.
#include "common.h"

namespace dc {
namespace {

typedef unsigned short u16;
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kAttWaves = 7, kAttRows = 4;   // waves per SIMD, rows of z that a lane group requests together

template <bool kBf16>
__device__ __forceinline__ void load8(const void* base, size_t row, int H, int ll, float (&x)[8]) {
  if constexpr (kBf16) {
    const v4u r = reinterpret_cast<const v4u*>(base)[row * (size_t)(H >> 3) + ll];
    x[0] = __uint_as_float(r.x << 16);
    x[1] = __uint_as_float(r.x & 0xFFFF0000u);
    x[2] = __uint_as_float(r.y << 16);
    x[3] = __uint_as_float(r.y & 0xFFFF0000u);
    x[4] = __uint_as_float(r.z << 16);
    x[5] = __uint_as_float(r.z & 0xFFFF0000u);
    x[6] = __uint_as_float(r.w << 16);
    x[7] = __uint_as_float(r.w & 0xFFFF0000u);
  } else {
    const float4* p = reinterpret_cast<const float4*>(base) + row * (size_t)(H >> 2) + 2 * ll;
    const float4 a = p[0], b = p[1];
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
  }
}

// s[v][k] = a_src^k . z^k_v and t[v][k] = a_dst^k . z^k_v for every node v and head k.
template <bool kBf16>
__global__ __launch_bounds__(256) void attention_scores_kernel(const void* __restrict__ z, int H, int K,
                                                                const float* __restrict__ att,
                                                                float* __restrict__ sc_src, float* __restrict__ sc_dst,
                                                                int* __restrict__ ctr, const int* __restrict__ node_off, int C,
                                                                const int* __restrict__ status) {
  if (status[0] != 0) return;
  if (blockIdx.x == 0) ctr[threadIdx.x] = 0;     // the counters of the kernel that follows
  const int ntot = node_off[C];
  const int LPR = H >> 3, LPH = LPR / K;       // lanes per row, lanes per head
  const int lane = threadIdx.x & 63, sg = lane / LPR, ll = lane - sg * LPR;
  const int rows_per_wave = 64 / LPR;
  const long long wave0 = ((long long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const long long nwaves = ((long long)gridDim.x * blockDim.x) >> 6;
  float as[8], ad[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    as[i] = att[ll * 8 + i];
    ad[i] = att[H + ll * 8 + i];
  }
  for (long long r0 = wave0 * rows_per_wave; r0 < ntot; r0 += nwaves * rows_per_wave) {
    const long long v = r0 + sg;
    float ps = 0.f, pd = 0.f;
    if (v < ntot) {
      float x[8];
      load8<kBf16>(z, (size_t)v, H, ll, x);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        ps += as[i] * x[i];
        pd += ad[i] * x[i];
      }
    }
    for (int o = 1; o < LPH; o <<= 1) {          // the head's lanes are adjacent and LPH-aligned
      ps += __shfl_xor(ps, o, 64);
      pd += __shfl_xor(pd, o, 64);
    }
    if (v < ntot && (ll % LPH) == 0) {
      sc_src[v * K + ll / LPH] = ps;
      sc_dst[v * K + ll / LPH] = pd;
    }
  }
}

// e_i = ReLU(sum over j in N_i of gamma_ij z_j + b): one group of LPR lanes per node, the list (i, predecessors,
// successors) in batches of LPH = H / (8 K) neighbours, for LPH >= 4.  Each of a head's LPH lanes takes one neighbour
// of the batch: its number, its score and the exponential are formed once per (neighbour, head) and handed round
// when the rows are summed; the running maximum and the rescaling of the partial sums happen once per batch.
// What bounds it is the way behind L2: the rows in work on an XCD and the rows their lists name have to stay in its
// 4 MB.  So rows are claimed in order (below) and results are stored past L2.  1.39 M rows, H = 256, four heads, per
// layer: 673 us and 23 M lines missed when every lane walked its list in rows dealt by a fixed stride, 612 us and 17 M
// with claims, 587 us with the stores as well.
template <bool kBf16>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kBf16 ? kAttWaves : 5, 8))) void attention_aggregate_kernel(
    const void* __restrict__ z, int H, int K, const float* __restrict__ sc_src, const float* __restrict__ sc_dst,
    const float* __restrict__ bias, const int* __restrict__ in_rp, const int* __restrict__ in_ci,
    const int* __restrict__ out_rp, const int* __restrict__ out_ci, void* __restrict__ out, int* __restrict__ ctr,
    const int* __restrict__ node_off, int C, const int* __restrict__ status) {
  if (status[0] != 0) return;
  const int ntot = node_off[C];
  const int LPR = H >> 3, LPH = LPR / K;
  const int lane = threadIdx.x & 63, sg = lane / LPR, ll = lane - sg * LPR;
  const int head = ll / LPH, li = ll - head * LPH, hb = lane - li;      // hb: the first of the head's lanes
  const int rows_per_wave = 64 / LPR;
  // Workgroups are dealt round-robin to the eight XCDs, each with its own L2: every XCD takes one contiguous eighth of
  // the rows, and its waves claim them in order, a few at a time, through a counter.  Dealt by a fixed stride the waves
  // drift apart, the rows in work span more than the L2, and neighbours' rows come from memory several times.
  const int xcd = blockIdx.x & 7;
  const int r_begin = (int)((long long)ntot * xcd / 8), r_end = (int)((long long)ntot * (xcd + 1) / 8);
  const int n_waves = (int)((gridDim.x >> 3) * (blockDim.x >> 6));
  // Claims of four rounds of rows (two where a round has 16) where every wave has sixteen rounds or more; below that
  // nothing drifts far and coarse claims leave waves idle at the end (80 k rows, H = 256: 269 us a pass with claims, 187
  // without), so the waves take single rounds in turn.
  const bool claims = r_end - r_begin >= 16 * n_waves * rows_per_wave;
  const int iters = !claims ? 1 : (rows_per_wave >= 16 ? 2 : 4);
  const int per_claim = rows_per_wave * iters;
  const int n_claims = (r_end - r_begin + per_claim - 1) / per_claim;
  int* my_ctr = ctr + xcd * 32;
  constexpr int U = kBf16 ? kAttRows : 4;        // rows requested together
  int cur = (int)((blockIdx.x >> 3) * (blockDim.x >> 6)) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  while (cur < n_claims) {
    int after = cur + n_waves;                                   // the first claim of a wave is its own number
    if (claims && lane == 0) after = n_waves + atomicAdd(my_ctr, 1);
    const int v0 = r_begin + cur * per_claim, nrows = min(per_claim, r_end - v0);
    // bounds of all rows of the claim (lane i: of row v0 + i), then the first 64 neighbour numbers of each direction
    const int rpi = in_rp[min(v0 + min(lane, per_claim), r_end)], rpo = out_rp[min(v0 + min(lane, per_claim), r_end)];
    const int ei = __builtin_amdgcn_readlane(rpi, 0), eo = __builtin_amdgcn_readlane(rpo, 0);
    const int ni = __builtin_amdgcn_readfirstlane(__shfl(rpi, per_claim, 64)) - ei;
    const int no = __builtin_amdgcn_readfirstlane(__shfl(rpo, per_claim, 64)) - eo;
    const int idi = *(ni > 0 ? in_ci + ei + min(lane, ni - 1) : in_rp);
    const int ido = *(no > 0 ? out_ci + eo + min(lane, no - 1) : in_rp);
    for (int it = 0; it < iters; ++it) {
    if (it * rows_per_wave >= nrows) break;
    const int rw = it * rows_per_wave + sg, rr = min(rw, nrows - 1), row = v0 + rr;   // rows past the end repeat the last
    const bool mine = rw < nrows;
    const int is = __shfl(rpi, rr, 64), din = __shfl(rpi, rr + 1, 64) - is;
    const int os = __shfl(rpo, rr, 64), n = 1 + din + __shfl(rpo, rr + 1, 64) - os;
    const float si = sc_src[(size_t)row * K + head];
    int id_first;
    {
      const int q = min(li, min(LPH, n) - 1);                    // position in N_i; lanes past the end repeat the last one
      const int pi = is - ei + q - 1, po = os - eo + q - 1 - din;
      const int x = __shfl(idi, max(pi, 0) & 63, 64), y = __shfl(ido, max(po, 0) & 63, 64);
      id_first = q == 0 ? row : (q <= din ? x : y);
      if (q > 0 && (q <= din ? pi : po) >= 64) {
        id_first = q <= din ? in_ci[ei + pi] : out_ci[eo + po];
        asm volatile("" : "+v"(id_first));                       // waited for here, not on the usual way as well
      }
    }
    float m = -INFINITY, den = 0.f;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int b0 = 0; b0 < n; b0 += LPH) {
      const int nb = min(LPH, n - b0);
      int id = id_first;
      if (b0 > 0) {
        const int q = b0 + min(li, nb - 1);
        id = q <= din ? in_ci[is + q - 1] : out_ci[os + q - 1 - din];
      }
      const float tj = sc_dst[(size_t)id * K + head];
      float p = 0.f, scale = 0.f;
      for (int k = 0; k < nb; k += U) {
        v4u xr[kBf16 ? U : 2 * U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int idu = __shfl(id, hb + min(k + u, nb - 1), 64);
          // past the end the last one again: a request in a branch would make every wait one for all requests
          if constexpr (kBf16) {
            xr[u] = reinterpret_cast<const v4u*>(z)[(size_t)idu * LPR + ll];
          } else {
            const v4u* zp = reinterpret_cast<const v4u*>(z) + (size_t)idu * (2 * LPR) + 2 * ll;
            xr[2 * u] = zp[0];
            xr[2 * u + 1] = zp[1];
          }
        }
        if (k == 0) {
          float e = si + tj;
          e = e > 0.f ? e : 0.2f * e;
          float mn = fmaxf(m, e);                 // lanes past the end repeat a neighbour: the maximum is the same
          for (int o = 1; o < LPH; o <<= 1) mn = fmaxf(mn, __shfl_xor(mn, o, 64));
          scale = __expf(m - mn);                 // 0 in the first batch (m = -inf)
          p = li < nb ? __expf(e - mn) : 0.f;
          m = mn;
          den = den * scale + p;                  // of this lane's neighbours; the head's lanes are added at the end
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[i] *= scale;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float pu = __shfl(p, hb + min(k + u, nb - 1), 64);
          if (k + u < nb) {
            if constexpr (kBf16) {
              const unsigned w[4] = {xr[u].x, xr[u].y, xr[u].z, xr[u].w};
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                acc[2 * i] += pu * __uint_as_float(w[i] << 16);
                acc[2 * i + 1] += pu * __uint_as_float(w[i] & 0xFFFF0000u);
              }
            } else {
              const unsigned w[8] = {xr[2 * u].x,     xr[2 * u].y,     xr[2 * u].z,     xr[2 * u].w,
                                     xr[2 * u + 1].x, xr[2 * u + 1].y, xr[2 * u + 1].z, xr[2 * u + 1].w};
#pragma unroll
              for (int i = 0; i < 8; ++i) acc[i] += pu * __uint_as_float(w[i]);
            }
          }
        }
      }
    }
    for (int o = 1; o < LPH; o <<= 1) den += __shfl_xor(den, o, 64);
    if (!mine) continue;
    const float inv = 1.0f / den;                 // N_i holds at least i itself
    float y[8];
    {
      const float4 b0 = *reinterpret_cast<const float4*>(bias + ll * 8);        // read here, not kept across
      const float4 b1 = *reinterpret_cast<const float4*>(bias + ll * 8 + 4);    // the walk: registers are scarce
      y[0] = fmaxf(acc[0] * inv + b0.x, 0.f);
      y[1] = fmaxf(acc[1] * inv + b0.y, 0.f);
      y[2] = fmaxf(acc[2] * inv + b0.z, 0.f);
      y[3] = fmaxf(acc[3] * inv + b0.w, 0.f);
      y[4] = fmaxf(acc[4] * inv + b1.x, 0.f);
      y[5] = fmaxf(acc[5] * inv + b1.y, 0.f);
      y[6] = fmaxf(acc[6] * inv + b1.z, 0.f);
      y[7] = fmaxf(acc[7] * inv + b1.w, 0.f);
    }
    if constexpr (kBf16) {
      v4u o;
      o.x = pack_bf16x2(y[0], y[1]);
      o.y = pack_bf16x2(y[2], y[3]);
      o.z = pack_bf16x2(y[4], y[5]);
      o.w = pack_bf16x2(y[6], y[7]);
      __builtin_nontemporal_store(o, reinterpret_cast<v4u*>(out) + (size_t)row * LPR + ll);   // L2 is for z
    } else {
      float4* p = reinterpret_cast<float4*>(out) + (size_t)row * (H >> 2) + 2 * ll;
      p[0] = make_float4(y[0], y[1], y[2], y[3]);
      p[1] = make_float4(y[4], y[5], y[6], y[7]);
    }
    }
    cur = __builtin_amdgcn_readfirstlane(after);
  }
}

// The same for heads of one or two lanes (LPH < 4): one group of LPR lanes per node walks
// the list (i, predecessors, successors) once, keeping a running maximum of the scores and
// rescaling the partial sums when it grows (the usual single-pass softmax), fp32 throughout.
// The group's lanes fetch up to LPR neighbour ids in one load and hand them round; rows and
// score terms of four neighbours are in flight at a time.  Held to 64 registers so that eight
// waves share a SIMD: the walk is a chain of dependent loads and only occupancy hides it.
template <bool kBf16>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8))) void attention_aggregate_walk_kernel(
    const void* __restrict__ z, int H, int K, const float* __restrict__ sc_src, const float* __restrict__ sc_dst,
    const float* __restrict__ bias, const int* __restrict__ in_rp, const int* __restrict__ in_ci,
    const int* __restrict__ out_rp, const int* __restrict__ out_ci, void* __restrict__ out,
    const int* __restrict__ node_off, int C, const int* __restrict__ status) {
  if (status[0] != 0) return;
  const int ntot = node_off[C];
  const int LPR = H >> 3, LPH = LPR / K;
  const int lane = threadIdx.x & 63, sg = lane / LPR, ll = lane - sg * LPR, hb = sg * LPR;
  const int head = ll / LPH;
  const int rows_per_wave = 64 / LPR, rows_per_wg = rows_per_wave * (blockDim.x >> 6);
  // Workgroups are dealt round-robin to the eight XCDs, each with its own L2: every XCD takes
  // one contiguous eighth of the rows, so that the neighbours of its rows (a graph is a few
  // hundred KB of z) are fetched into one L2 only.  The grid is a multiple of 8 workgroups.
  const long long n_chunks = (ntot + rows_per_wg - 1) / rows_per_wg;
  const int xcd = blockIdx.x & 7, jx = blockIdx.x >> 3, per_x = gridDim.x >> 3;
  const long long c_begin = n_chunks * xcd / 8, c_end = n_chunks * (xcd + 1) / 8;
  for (long long chunk = c_begin + jx; chunk < c_end; chunk += per_x) {
    const long long v = chunk * rows_per_wg + (threadIdx.x >> 6) * rows_per_wave + sg;
    if (v >= ntot) continue;                     // whole lane groups drop out together
    const int is = in_rp[v], din = in_rp[v + 1] - is;
    const int os = out_rp[v], dout = out_rp[v + 1] - os;
    const int n = 1 + din + dout;
    const float si = sc_src[v * K + head];
    float m = -INFINITY, den = 0.f;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int b0 = 0; b0 < n; b0 += LPR) {
      const int nb = min(LPR, n - b0);
      int mine = 0;
      {
        const int q = b0 + ll;                    // position in N_i
        if (ll < nb) mine = q == 0 ? (int)v : (q <= din ? in_ci[is + q - 1] : out_ci[os + q - 1 - din]);
      }
      for (int k = 0; k < nb; k += 4) {
        int id[4];
        float tj[4], x[4][8];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          id[u] = __shfl(mine, hb + min(k + u, nb - 1), 64);       // past the end: repeats the last one, unused
          tj[u] = sc_dst[(size_t)id[u] * K + head];
          load8<kBf16>(z, (size_t)id[u], H, ll, x[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (k + u < nb) {
            float e = si + tj[u];
            e = e > 0.f ? e : 0.2f * e;
            const float mn = fmaxf(m, e);
            const float scale = __expf(m - mn);   // 0 at the first neighbour (m = -inf)
            const float p = __expf(e - mn);
            den = den * scale + p;
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] = acc[i] * scale + p * x[u][i];
            m = mn;
          }
        }
      }
    }
    const float inv = 1.0f / den;                 // N_i holds at least i itself
    float y[8];
    {
      const float4 b0 = *reinterpret_cast<const float4*>(bias + ll * 8);        // read here, not kept across
      const float4 b1 = *reinterpret_cast<const float4*>(bias + ll * 8 + 4);    // the walk: registers are scarce
      y[0] = fmaxf(acc[0] * inv + b0.x, 0.f);
      y[1] = fmaxf(acc[1] * inv + b0.y, 0.f);
      y[2] = fmaxf(acc[2] * inv + b0.z, 0.f);
      y[3] = fmaxf(acc[3] * inv + b0.w, 0.f);
      y[4] = fmaxf(acc[4] * inv + b1.x, 0.f);
      y[5] = fmaxf(acc[5] * inv + b1.y, 0.f);
      y[6] = fmaxf(acc[6] * inv + b1.z, 0.f);
      y[7] = fmaxf(acc[7] * inv + b1.w, 0.f);
    }
    if constexpr (kBf16) {
      v4u o;
      o.x = pack_bf16x2(y[0], y[1]);
      o.y = pack_bf16x2(y[2], y[3]);
      o.z = pack_bf16x2(y[4], y[5]);
      o.w = pack_bf16x2(y[6], y[7]);
      reinterpret_cast<v4u*>(out)[(size_t)v * LPR + ll] = o;
    } else {
      float4* p = reinterpret_cast<float4*>(out) + (size_t)v * (H >> 2) + 2 * ll;
      p[0] = make_float4(y[0], y[1], y[2], y[3]);
      p[1] = make_float4(y[4], y[5], y[6], y[7]);
    }
  }
}

}  // namespace

bool attention_shape_supported(int H, int heads) {
  const bool pow2_h = H >= 32 && H <= 512 && (H & (H - 1)) == 0;
  const bool pow2_k = heads >= 1 && (heads & (heads - 1)) == 0;
  return pow2_h && pow2_k && H / heads >= 8;
}

hipError_t launch_attention_scores(const GnnArgs& a, const void* z, const float* att_l, hipStream_t s) {
  const dim3 grid(a.n_cu * 8), block(256);
  if (a.bf16)
    hipLaunchKernelGGL(attention_scores_kernel<true>, grid, block, 0, s, z, a.H, a.heads, att_l, a.score[0],
                       a.score[1], a.heavy_ctr, a.node_off, a.n_cand, a.status);
  else
    hipLaunchKernelGGL(attention_scores_kernel<false>, grid, block, 0, s, z, a.H, a.heads, att_l, a.score[0],
                       a.score[1], a.heavy_ctr, a.node_off, a.n_cand, a.status);
  return hipGetLastError();
}

hipError_t launch_attention_aggregate(const GnnArgs& a, const void* z, const float* bias, void* out, hipStream_t s) {
  // batches of fewer than four neighbours would leave too few rows in flight
  const bool batches = a.H / (8 * a.heads) >= 4;
  const dim3 block(256);                        // every workgroup resident from the start
  if (batches) {
    static_assert(kHeavyCtrInts == 256, "attention_scores_kernel clears one counter word per thread");
    const dim3 grid(((a.n_cu + 7) / 8) * 8 * (a.bf16 ? kAttWaves : 5));
    auto kern = a.bf16 ? attention_aggregate_kernel<true> : attention_aggregate_kernel<false>;
    hipLaunchKernelGGL(kern, grid, block, 0, s, z, a.H, a.heads, a.score[0], a.score[1], bias, a.in_rowptr, a.in_col,
                       a.out_rowptr, a.out_col, out, a.heavy_ctr, a.node_off, a.n_cand, a.status);
  } else {
    auto kern = a.bf16 ? attention_aggregate_walk_kernel<true> : attention_aggregate_walk_kernel<false>;
    hipLaunchKernelGGL(kern, dim3(((a.n_cu + 7) / 8) * 8 * 8), block, 0, s, z, a.H, a.heads, a.score[0], a.score[1], bias,
                       a.in_rowptr, a.in_col, a.out_rowptr, a.out_col, out, a.node_off, a.n_cand, a.status);
  }
  return hipGetLastError();
}

}  // namespace dc
