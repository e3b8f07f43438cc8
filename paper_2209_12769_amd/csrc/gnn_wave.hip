// Message-passing layer for the narrower bf16 shapes (input width 16, 32, 64 or, for outputs wider than 32, 128; output
// width 32, 64 or 128; gfx950):
//     h'[v] = ReLU([h[v] | mean_pred(h)[v] | mean_succ(h)[v]] W + b)
// One pass over the rows; neither mean is written to HBM.
//
// What bounds it is the latency of row pointers -> neighbour numbers -> neighbour rows, not bandwidth or the matrix
// cores (1.1 M rows at 128 x 128 are 0.6 GB and 0.1 TFLOP).  So no wave ever waits for another one: all of W lies in
// LDS for the workgroup's life (96 KB at 128 x 128, loaded once), every wave takes tiles of 32 rows of its own, forms
// their means in registers, turns them into matrix operands through 32 rows of LDS that only it uses, and multiplies
// all output columns.  The neighbours of up to four row groups are in flight at any time, across the ends of a
// direction and of a tile; pointers and neighbour numbers come a tile ahead.
// 1.1 M rows, 128 -> 128 columns: 436 us (607 with four waves per 128-row tile, two barriers per 64 columns and a serial
// walk over neighbours three and up); 32 -> 128: 168 us (225 as separate aggregate and update).  With requests inside
// branches, where the compiler's waits drain everything, the same structure took 560 us.
#include "common.h"

namespace dc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned short u16;
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kWT = 512;            // threads per workgroup: two waves per SIMD, 256 registers each
constexpr int kTR = 32;             // rows per wave and tile
constexpr int kSlots = 5;           // neighbours per row and direction that are requested together

template <int D, int H>
struct WaveShape {
  static constexpr int WBytes = 3 * D * H * 2;
  static constexpr int PassCols = H > 64 && D <= 64 ? 64 : H;       // columns that are written out together
  static constexpr int AreaBytes = kTR * (D > PassCols ? D : PassCols) * 2;
  static constexpr int Lds = WBytes + (kWT / 64) * AreaBytes;
  static constexpr int PerCu = D * H <= 1024 ? 2 : 1;               // what the kernel's registers allow
  static_assert(Lds <= 160 * 1024, "W and the waves' areas share one CU's LDS");
};

// Index of 16-byte piece c of row r in an area with P pieces per row: XOR-swizzled so that 32 lanes that read the same
// piece of 32 rows hit every bank equally.
template <int P>
__device__ __forceinline__ int swz(int r, int c) {
  return r * P + (c ^ ((r / (16 / P)) & (P - 1)));
}

__device__ __forceinline__ void set8(float* acc, const v4u x) {   // first neighbour: exact unpack
  acc[0] = __uint_as_float(x.x << 16);
  acc[1] = __uint_as_float(x.x & 0xFFFF0000u);
  acc[2] = __uint_as_float(x.y << 16);
  acc[3] = __uint_as_float(x.y & 0xFFFF0000u);
  acc[4] = __uint_as_float(x.z << 16);
  acc[5] = __uint_as_float(x.z & 0xFFFF0000u);
  acc[6] = __uint_as_float(x.w << 16);
  acc[7] = __uint_as_float(x.w & 0xFFFF0000u);
}
__device__ __forceinline__ void add8(float* acc, const v4u x, unsigned one) {   // further neighbours
  bf16_pair_add(acc[0], acc[1], x.x, one);
  bf16_pair_add(acc[2], acc[3], x.y, one);
  bf16_pair_add(acc[4], acc[5], x.z, one);
  bf16_pair_add(acc[6], acc[7], x.w, one);
}

// LDS that one wave writes and reads needs no barrier, only that the compiler keeps the order.
__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

// The same value, as one the compiler cannot compute addresses from ahead of the loop (kept there they cost dozens of
// registers).
__device__ __forceinline__ int here(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Row pointers (lane i <= 32: of row m0 + i) and the first 128 neighbour numbers of a tile and direction.
struct Lists {
  int rp, id0, id1;
};

extern __shared__ __attribute__((aligned(16))) char dc_wave_smem[];

template <int D, int H>
__global__ __launch_bounds__(kWT) void wave_layer_kernel(const u16* __restrict__ h, const int* __restrict__ in_rp,
                                                         const int* __restrict__ in_ci, const int* __restrict__ out_rp,
                                                         const int* __restrict__ out_ci, const u16* __restrict__ Wp,
                                                         const float* __restrict__ bias, u16* __restrict__ out,
                                                         const int* __restrict__ node_off, int C,
                                                         const int* __restrict__ status) {
  using S = WaveShape<D, H>;
  constexpr int P = D / 8, RPI = 64 / P, NG = kTR / RPI;    // lanes per row, rows per load, loads per tile
  constexpr int R = NG < 4 ? NG : 4;                       // row groups whose neighbours are in flight at a time
  constexpr int PO = S::PassCols / 8, RPO = 64 / PO, TN = H / 32, TP = S::PassCols / 32;
  if (status[0] != 0) return;
  const int ntot = node_off[C];
  const int ntiles = (ntot + kTR - 1) / kTR;
  // Workgroups are dealt round-robin to the eight XCDs: each takes one contiguous eighth of the tiles, so that
  // neighbours' rows are fetched into one L2.  Within it workgroups first, waves second: few tiles spread over CUs.
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, per = gridDim.x >> 3;
  const int tpx = (ntiles + 7) >> 3;
  const int t_end = min(ntiles, (xcd + 1) * tpx);
  if (xcd * tpx + slot >= t_end) return;                   // none of its waves has a tile

  v4u* Ws = reinterpret_cast<v4u*>(dc_wave_smem);          // [3 D / 8][H] pieces, as packed in memory
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  v4u* area = reinterpret_cast<v4u*>(dc_wave_smem + S::WBytes + wave * S::AreaBytes);
  {
    const v4u* wsrc = reinterpret_cast<const v4u*>(Wp);
#pragma unroll
    for (int i = 0; i < (3 * D * H / 8 + kWT - 1) / kWT; ++i)
      if (t + i * kWT < 3 * D * H / 8) Ws[t + i * kWT] = wsrc[t + i * kWT];
  }
  __syncthreads();

  const int l32 = lane & 31, lh = lane >> 5;
  const int sub = lane / P, piece = lane % P;
  const v4u* __restrict__ h4 = reinterpret_cast<const v4u*>(h);
  const unsigned one = bf16_one_reg();

  auto load_rp = [&](const int* rp, int tile) __attribute__((always_inline)) {
    return rp[min(tile * kTR + min(lane, kTR), ntot)];
  };
  auto load_ids = [&](const int* ci, Lists& l) __attribute__((always_inline)) {
    const int e0 = __builtin_amdgcn_readlane(l.rp, 0), e1 = __builtin_amdgcn_readlane(l.rp, kTR);
    // a tile without neighbours takes number 0, which node_off begins with (a caller's row pointers may begin anywhere)
    const int* q0 = e1 > e0 ? ci + min(e0 + lane, e1 - 1) : node_off;
    const int* q1 = e1 > e0 ? ci + min(e0 + 64 + lane, e1 - 1) : node_off;
    l.id0 = *q0;
    l.id1 = *q1;
  };
  // neighbour number at place p of the tile's list (all lanes take part; p < 0: don't care)
  auto id_at = [&](const int* ci, const Lists& l, int e0, int p) __attribute__((always_inline)) {
    const int a = __shfl(l.id0, p & 63, 64), b = __shfl(l.id1, p & 63, 64);
    int id = p < 64 ? a : b;
    if (p >= 128) {
      id = ci[e0 + p];
      asm volatile("" : "+v"(id));                         // waited for here, not on the usual way as well
    }
    return id;
  };
  // No request below stands in a branch (what does not exist repeats something that does): the compiler counts
  // outstanding requests, and behind a branch that may have made none it waits for all of them.
  // One row group and direction in flight: places of the lists, lengths, up to kSlots neighbours' pieces
  struct Unit {
    int ps, dg;
    v4u x[kSlots];
  } un[R];
  v4u xs[NG];
  auto issue_self = [&](int tile) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int row = min(tile * kTR + g * RPI + sub, ntot - 1);
      xs[g] = h4[(size_t)row * P + piece];
    }
  };
  auto issue = [&](Unit& w, const int* ci, const Lists& l, int g) __attribute__((always_inline)) {
    const int e0 = __builtin_amdgcn_readlane(l.rp, 0), r = g * RPI + sub;
    const int s = __shfl(l.rp, r, 64);
    w.dg = __shfl(l.rp, r + 1, 64) - s;
    w.ps = s - e0;
    int id[kSlots];
#pragma unroll
    for (int k = 0; k < kSlots; ++k) id[k] = id_at(ci, l, e0, w.dg > 0 ? w.ps + min(k, w.dg - 1) : 0);
#pragma unroll
    for (int k = 0; k < kSlots; ++k) w.x[k] = h4[(size_t)id[k] * P + piece];
  };
  // the means of a row group, as operands in the wave's area; neighbours beyond kSlots eight at a time
  auto reduce = [&](const Unit& w, const int* ci, const Lists& l, int g) __attribute__((always_inline)) {
    const int e0 = __builtin_amdgcn_readlane(l.rp, 0);
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    if (w.dg > 0) set8(acc, w.x[0]);
#pragma unroll
    for (int k = 1; k < kSlots; ++k)
      if (w.dg > k) add8(acc, w.x[k], one);
    for (int u = kSlots; __any(w.dg > u); u += 8) {
      v4u y[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        y[k] = h4[(size_t)id_at(ci, l, e0, w.dg > u ? w.ps + min(u + k, w.dg - 1) : 0) * P + piece];
      }
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (w.dg > u + k) add8(acc, y[k], one);
    }
    const float sc = w.dg > 0 ? 1.0f / (float)w.dg : 0.0f;
    v4u o;
    o.x = pack_bf16x2(acc[0] * sc, acc[1] * sc);
    o.y = pack_bf16x2(acc[2] * sc, acc[3] * sc);
    o.z = pack_bf16x2(acc[4] * sc, acc[5] * sc);
    o.w = pack_bf16x2(acc[6] * sc, acc[7] * sc);
    area[swz<P>(g * RPI + sub, piece)] = o;
  };
  // all row groups of one direction; the units they free go to the groups R further on, in the end of the next part
  auto means = [&](const int* ci, const Lists& l, const int* ci_next, const Lists& l_next) __attribute__((always_inline)) {
#pragma unroll 1
    for (int b = 0; b < NG - R; b += R)
#pragma unroll
      for (int j = 0; j < R; ++j) {
        reduce(un[j], ci, l, b + j);
        issue(un[j], ci, l, b + R + j);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      reduce(un[j], ci, l, NG - R + j);
      issue(un[j], ci_next, l_next, j);
      __builtin_amdgcn_sched_barrier(0);
    }
    wave_order();
  };
  f32x16 acc[TN];
  // operands swapped: the accumulator tile is (column, row), so a lane owns one row and four consecutive columns per
  // register quad
  auto multiply = [&](int seg) __attribute__((always_inline)) {
    const int lr = here(l32);
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      const bf16x8 a = __builtin_bit_cast(bf16x8, area[swz<P>(lr, 2 * ks + lh)]);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const bf16x8 b = __builtin_bit_cast(bf16x8, Ws[(seg * P + 2 * ks + lh) * H + j * 32 + l32]);
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, acc[j], 0, 0, 0);
      }
    }
    wave_order();
  };

  int tile = xcd * tpx + slot + wave * per;
  const int step = per * (kWT / 64);
  if (tile >= t_end) return;
  Lists li, lo;
  li.rp = load_rp(in_rp, tile);
  lo.rp = load_rp(out_rp, tile);
  issue_self(tile);
  load_ids(in_ci, li);
  load_ids(out_ci, lo);
#pragma unroll
  for (int j = 0; j < R; ++j) issue(un[j], in_ci, li, j);
  for (;;) {
    const int next = tile + step;
    const bool more = next < t_end;                        // the wave's last tile requests itself once more
    const int tn = more ? next : tile;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    Lists ni, no;
    ni.rp = load_rp(in_rp, tn);
    no.rp = load_rp(out_rp, tn);
#pragma unroll
    for (int g = 0; g < NG; ++g) area[swz<P>(g * RPI + sub, piece)] = xs[g];
    wave_order();
    multiply(0);
    means(in_ci, li, out_ci, lo);
    load_ids(in_ci, ni);
    load_ids(out_ci, no);
    multiply(1);
    means(out_ci, lo, in_ci, ni);
    issue_self(tn);
    __builtin_amdgcn_sched_barrier(0);
    multiply(2);
    // bias, ReLU, bf16, whole rows through the wave's area
    const float* bp = bias;
    asm volatile("" : "+s"(bp));                           // read here, by scalar loads, not kept in 64 registers
    const int lq = here(l32), le = here(lane);
#pragma unroll
    for (int pass = 0; pass < H / S::PassCols; ++pass) {
#pragma unroll
      for (int jj = 0; jj < TP; ++jj)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int j = pass * TP + jj;
          float y[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float lo = bp[j * 32 + 8 * q + i], hi = bp[j * 32 + 8 * q + 4 + i];
            y[i] = fmaxf(acc[j][4 * q + i] + (lh ? hi : lo), 0.f);
          }
          uint2 p;
          p.x = pack_bf16x2(y[0], y[1]);
          p.y = pack_bf16x2(y[2], y[3]);
          reinterpret_cast<uint2*>(area)[2 * swz<PO>(lq, jj * 4 + q) + lh] = p;
        }
      wave_order();
#pragma unroll
      for (int i = 0; i < kTR / RPO; ++i) {
        const int r = min(i * RPO + le / PO, ntot - 1 - tile * kTR), c = le % PO;     // beyond the end: the last row again
        reinterpret_cast<v4u*>(out)[(size_t)(tile * kTR + r) * (H / 8) + pass * PO + c] = area[swz<PO>(r, c)];
      }
      wave_order();
    }
    if (!more) break;
    tile = next;
    li = ni;
    lo = no;
  }
}

template <int D, int H>
hipError_t launch(const GnnArgs& a, const void* h, const void* Wl, const float* bias, void* out, hipStream_t s) {
  using S = WaveShape<D, H>;
  auto kern = wave_layer_kernel<D, H>;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, S::Lds);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3(((a.n_cu * S::PerCu + 7) / 8) * 8), dim3(kWT), S::Lds, s, static_cast<const u16*>(h),
                     a.in_rowptr, a.in_col, a.out_rowptr, a.out_col, static_cast<const u16*>(Wl), bias,
                     static_cast<u16*>(out), a.node_off, a.n_cand, a.status);
  return hipGetLastError();
}

template <int H>
hipError_t launch_width(int d, const GnnArgs& a, const void* h, const void* Wl, const float* bias, void* out,
                        hipStream_t s) {
  if (d == 16) return launch<16, H>(a, h, Wl, bias, out, s);
  if (d == 32) return launch<32, H>(a, h, Wl, bias, out, s);
  if constexpr (H > 32) {
    if (d == 128) return launch<128, H>(a, h, Wl, bias, out, s);
  }
  return launch<64, H>(a, h, Wl, bias, out, s);
}

}  // namespace

// Widths whose three blocks of W fit LDS beside the waves' areas and whose rows divide a wave's lanes.
bool wave_layer_supported(int d, int H, int bf16) {
  return bf16 && (d == 16 || d == 32 || d == 64 || (d == 128 && H > 32)) && (H == 32 || H == 64 || H == 128);
}

hipError_t launch_wave_layer(const void* h, int d, const GnnArgs& a, const void* Wl, const float* bias, void* out,
                             hipStream_t s) {
  if (a.H == 32) return launch_width<32>(d, a, h, Wl, bias, out, s);
  if (a.H == 64) return launch_width<64>(d, a, h, Wl, bias, out, s);
  return launch_width<128>(d, a, h, Wl, bias, out, s);
}

}  // namespace dc
