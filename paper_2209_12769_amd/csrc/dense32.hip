// Products of fp32 matrices on the bf16 matrix cores: out = [A0 | A1 | A2] W (+ bias, ReLU), gfx950.
//
// An fp32 number of 2^-110 to 3.39e38 is exactly the sum of three bf16 numbers (8 + 8 + 8 bits of its significand: x1 = bf16(x),
// x2 = bf16(x - x1), x3 = x - x1 - x2; both differences are exact).  Below, the third piece falls under bf16's smallest number,
// 2^-133, and what is lost is at most that.  Of the nine partial products the six with i + j <= 4 are formed; each is exact in
// fp32 unless it lies below fp32's smallest numbers, and what is left out (x2 w3, x3 w2, x3 w3) is below 2^-25 of |x w|, less
// than the rounding of one fp32 addition.
// Why: mfma_f32_32x32x2f32 takes 64 cycles for 2 rows of W, mfma_f32_32x32x16_bf16 32 cycles for 16: six of the latter
// do in 192 cycles what eight of the former do in 512.
// Sums: the matrix cores align the 16 products of an instruction to the largest one and drop what lies more than 24
// bits below it, downwards (towards minus infinity), then add to the accumulator with one rounding to nearest (measured).  Two
// things follow.  The rows of W are taken in sections of 64, each into an accumulator of its own that is added to the
// total by the vector ALU: the total is rounded 12 times at K = 768 instead of 288 (384 with the fp32 instructions).  And
// every other section's W is stored negated and its sum subtracted: what is dropped cancels.  The small partial products
// of a chunk come first, so that a section's first chunk is rounded once at its full size.  Against 64-bit sums of
// inputs like those of the layers (ReLU outputs, normal weights), error over the root mean square of the result: K = 48
// 0.99e-7 (fp32 instructions 0.98e-7), 96 1.04e-7 (1.40e-7), 192 1.16e-7 (1.76e-7), 384 1.23e-7 (2.64e-7), 768 1.26e-7 (3.39e-7);
// positive operands: 48 0.72e-7 (1.03e-7), 768 0.62e-7 (4.04e-7).
// Measured: 475 k rows, K = 256, 768 columns: 1.62 ms with the fp32 instructions, 1.22 ms; 96 k rows, K = 384, 128 columns
// 105 -> 70 us; 475 k rows of weight gradients (768 x 256) 1.5 -> 1.05 ms; the reverse pass of those rows in all 9.6 -> 7.5 ms.
// The matrix cores are busy 43 % of the time at 2.1 GHz, 45 % in the weight gradients.
//
// The pieces of W are made once per set of weights (pack_split_kernel) and lie as the matrix instruction reads them:
// unit (chunk c of 16 rows, piece p, half h of the chunk, column n) = 8 consecutive rows = 16 bytes.  The pieces of A
// are made in registers.
//
// Numbers that are not finite, or so close to the largest fp32 number that their first piece rounds to infinity, give
// an output that is not finite; a wave that sees one computes its tile again with the fp32 instructions and takes
// from there the outputs that are not finite, so that one row's numbers do not change another's bits.
#include <type_traits>

#include "common.h"

namespace dc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned short u16;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct Pieces {
  u32x4 p[3];          // 8 values: first, second, third piece
};
struct Pair {
  unsigned p[3];       // two values
};
__device__ __forceinline__ Pair split2(float x, float y) {
  const unsigned a = pack_bf16x2(x, y);
  const float rx = x - __uint_as_float(a << 16), ry = y - __uint_as_float(a & 0xFFFF0000u);
  const unsigned b = pack_bf16x2(rx, ry);
  return {{a, b, pack_bf16x2(rx - __uint_as_float(b << 16), ry - __uint_as_float(b & 0xFFFF0000u))}};
}
__device__ __forceinline__ Pieces split8(const f32x4& u, const f32x4& v) {
  const Pair a = split2(u.x, u.y), b = split2(u.z, u.w), c = split2(v.x, v.y), d = split2(v.z, v.w);
  Pieces r;
#pragma unroll
  for (int p = 0; p < 3; ++p) r.p[p] = u32x4{a.p[p], b.p[p], c.p[p], d.p[p]};
  return r;
}
__device__ __forceinline__ bf16x8 as_bf16(const u32x4& x) { return __builtin_bit_cast(bf16x8, x); }

constexpr int kSection = 4;          // chunks of 16 rows of W
__device__ __forceinline__ float section_sign(int chunk) { return (chunk / kSection) & 1 ? -1.f : 1.f; }

// ---- the pieces of W, in the order the products read them ----
// element (k, n) of the matrix is src[k * ld + n], or src[n * ld + k] (transposed); plain: the matrix itself, row by row
__global__ __launch_bounds__(256) void pack_split_kernel(SplitJobs jobs) {
  const SplitJob j = jobs.job[blockIdx.y];
  const int units = j.K / 8 * j.N;                       // 8 rows of one column each
  u32x4* __restrict__ dst = reinterpret_cast<u32x4*>(j.dst);
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < units; i += gridDim.x * blockDim.x) {
    const int k8 = i / j.N, n = i - k8 * j.N;
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      x[u] = j.transposed ? j.src[(size_t)n * j.ld + k8 * 8 + u] : j.src[(size_t)(k8 * 8 + u) * j.ld + n];
    if (j.plain) {
      float* out = reinterpret_cast<float*>(j.dst) + (size_t)k8 * 8 * j.N + n;
#pragma unroll
      for (int u = 0; u < 8; ++u) out[(size_t)u * j.N] = x[u];
      continue;
    }
    const float sign = section_sign(k8 >> 1);
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] *= sign;
    const Pieces s = split8(f32x4{x[0], x[1], x[2], x[3]}, f32x4{x[4], x[5], x[6], x[7]});
#pragma unroll
    for (int p = 0; p < 3; ++p) dst[((size_t)(k8 >> 1) * 6 + p * 2 + (k8 & 1)) * j.N + n] = s.p[p];
  }
}

struct Operands {
  const float *A0, *A1, *A2;
  const u32x4* Ws;
  const float* Wf;
  const float* bias;
  float* out;
  int d, nseg, N, ntot;
  int wk, wn;            // element (k, n) of W is Wf[k * wk + n * wn]
};

// First column of chunk c of [A0 | A1 | A2] (16 columns each; past the end the last one).  No branches: behind one the
// compiler waits for every load, and keeps no order of instructions across it.
__device__ __forceinline__ const float* chunk_base(const Operands& o, int c) {
  const int per = o.d >> 4;
  c = min(c, o.nseg * per - 1);
  const int seg = (c >= per ? 1 : 0) + (c >= 2 * per ? 1 : 0);
  const size_t a0 = (size_t)o.A0, a1 = (size_t)o.A1, a2 = (size_t)o.A2;
  const size_t base = seg == 0 ? a0 : (seg == 1 ? a1 : a2);
  return reinterpret_cast<const float*>(base) + (c - seg * per) * 16;
}

// Accumulator register v of lane (l32 = lane & 31, lh = lane >> 5) holds column 8 (v / 4) + 4 lh + v % 4 of its block of
// 32 (W is the first operand of the instruction), row l32: four consecutive columns per lane and quad.
__device__ __forceinline__ void store_quad(const Operands& o, f32x4 y, int row, int col) {
  if (o.bias) {
    const f32x4 b = *reinterpret_cast<const f32x4*>(o.bias + col);
    y = f32x4{fmaxf(y.x + b.x, 0.f), fmaxf(y.y + b.y, 0.f), fmaxf(y.z + b.z, 0.f), fmaxf(y.w + b.w, 0.f)};
  }
  *reinterpret_cast<f32x4*>(o.out + (size_t)row * o.N + col) = y;
}
__device__ __forceinline__ void store_block(const Operands& o, const f32x16& acc, int row, int col0, int lh) {
  if (row >= o.ntot) return;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    store_quad(o, f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]}, row, col0 + 8 * q + 4 * lh);
}
// 0 where every value of the block is finite, else NaN
__device__ __forceinline__ float finite_probe(const f32x16& acc, float t) {
#pragma unroll
  for (int v = 0; v < 16; ++v) t = fmaf(acc[v], 0.f, t);
  return t;
}
// 32 rows from m0, 32 columns from n0, in fp32 instructions straight from memory
__device__ __forceinline__ f32x16 fp32_block(const Operands& o, int m0, int n0) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
  const size_t off = (size_t)min(m0 + l32, o.ntot - 1) * o.d + lh;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  const float* w = o.Wf + (size_t)lh * o.wk + (size_t)(n0 + l32) * o.wn;
  for (int seg = 0; seg < o.nseg; ++seg) {
    const float* a = (seg == 0 ? o.A0 : (seg == 1 ? o.A1 : o.A2)) + off;
    for (int k = 0; k < o.d; k += 2, w += 2 * (size_t)o.wk) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[0], a[k], acc, 0, 0, 0);
  }
  return acc;
}
// The block with the outputs that are not finite from fp32 instructions, the others as they are: rows of other candidates that
// share its tile keep the bits that they have without it.
__device__ __forceinline__ f32x16 mended(const f32x16& split, const f32x16& fp32) {
  f32x16 y;
#pragma unroll
  for (int v = 0; v < 16; ++v) y[v] = __builtin_isfinite(split[v]) ? split[v] : fp32[v];
  return y;
}

// The six products of a chunk and a block of 32 columns; sections and order are the same in every kernel of this file, so
// that a result does not depend on the size of its batch.
__device__ __forceinline__ f32x16 product(const u32x4& w, const u32x4& a, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16(w), as_bf16(a), c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int v = 0; v < 16; ++v) z[v] = 0.f;
  return z;
}
__device__ __forceinline__ void add_section(f32x16& total, const f32x16& acc, float sign) {
#pragma unroll
  for (int v = 0; v < 16; ++v) total[v] = fmaf(acc[v], sign, total[v]);
}

// ---------------------------------------------------------------------------
// few rows: one wave per 32 x 32 tile, operands straight from memory
// ---------------------------------------------------------------------------
// A 128-row tile keeps one CU's matrix cores busy for 8 us at K = 384 and 128 columns whether or not the other 255 CUs
// have work.  With at most one 32 x 32 tile per SIMD of the chip the product is spread over all of them: 2 us of
// products each, no LDS and no barriers, operands three chunks ahead in registers.
__device__ __forceinline__ bool few_tiles(int ntot, int N, int most) { return ((ntot + 31) >> 5) * (N >> 5) <= most; }

struct FewChunk {
  f32x4 a[2];
  u32x4 w[3];
};
__device__ __forceinline__ void few_fetch(const Operands& o, FewChunk& x, int c, size_t aoff, const u32x4* wp) {
  const float* a = chunk_base(o, c) + aoff;
  x.a[0] = *reinterpret_cast<const f32x4*>(a);
  x.a[1] = *reinterpret_cast<const f32x4*>(a + 4);
#pragma unroll
  for (int p = 0; p < 3; ++p) x.w[p] = (wp + (size_t)c * 6 * o.N)[(size_t)p * 2 * o.N];
}
template <int kInSection>
__device__ __forceinline__ void few_step(const Operands& o, f32x16& total, f32x16& acc, FewChunk& cur, FewChunk& free, int c,
                                         int nk, size_t aoff, const u32x4* wp) {
  if (c >= nk) return;
  few_fetch(o, free, min(c + 3, nk - 1), aoff, wp);
  __builtin_amdgcn_sched_barrier(0);                  // the requests stay ahead of the products
  const Pieces s = split8(cur.a[0], cur.a[1]);
  acc = product(cur.w[2], s.p[0], kInSection == 0 ? zero16() : acc);
  acc = product(cur.w[1], s.p[1], acc);
  acc = product(cur.w[1], s.p[0], acc);
  acc = product(cur.w[0], s.p[2], acc);
  acc = product(cur.w[0], s.p[1], acc);
  acc = product(cur.w[0], s.p[0], acc);
  if (kInSection == kSection - 1 || c == nk - 1) add_section(total, acc, section_sign(c));
  __builtin_amdgcn_sched_barrier(0);
}
// Fewer tiles still, at most one per workgroup of the grid: the four waves of a workgroup share a tile.  Wave w has sections
// w, w + 4 .. of W and leaves their sums in LDS; wave w then adds quad w of all sections in their order, which gives the
// bits that one wave gives.  `sums`: a section's 1024 sums each.  A search step's layers of some hundred rows, K = 384 and
// 128: 16.6 and 9.8 us with the fp32 instructions and one wave per tile, 5.9 us on average; the search 5.6 -> 4.9 ms.
__device__ __forceinline__ void update_fewer(const Operands& o, float* sums) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int l32 = lane & 31, lh = lane >> 5;
  const int nct = o.N >> 5, ntiles = ((o.ntot + 31) >> 5) * nct, nk = o.nseg * o.d / 16, nsec = (nk + kSection - 1) / kSection;
  const int tile = blockIdx.x;
  if (tile >= ntiles) return;
  const int m0 = (tile / nct) * 32, n0 = (tile % nct) * 32, row = m0 + l32;
  const size_t aoff = (size_t)min(row, o.ntot - 1) * o.d + 8 * lh;
  const u32x4* wp = o.Ws + (size_t)lh * o.N + n0 + l32;
  if (wave < nsec) {
    FewChunk x[kSection];
#pragma unroll
    for (int i = 0; i < kSection; ++i) few_fetch(o, x[i], min(wave * kSection + i, nk - 1), aoff, wp);
    for (int sec = wave; sec < nsec; sec += 4) {
      f32x16 acc = zero16();
#pragma unroll
      for (int i = 0; i < kSection; ++i) {
        const int c = sec * kSection + i;
        const Pieces s = split8(x[i].a[0], x[i].a[1]);
        const u32x4 w0 = x[i].w[0], w1 = x[i].w[1], w2 = x[i].w[2];
        few_fetch(o, x[i], min(c + 4 * kSection, nk - 1), aoff, wp);
        if (c < nk) {
          acc = product(w2, s.p[0], acc);
          acc = product(w1, s.p[1], acc);
          acc = product(w1, s.p[0], acc);
          acc = product(w0, s.p[2], acc);
          acc = product(w0, s.p[1], acc);
          acc = product(w0, s.p[0], acc);
        }
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) sums[(sec * 16 + v) * 64 + lane] = acc[v];
    }
  }
  __syncthreads();
  float y[4] = {0.f, 0.f, 0.f, 0.f};
  for (int sec = 0; sec < nsec; ++sec)
#pragma unroll
    for (int u = 0; u < 4; ++u) y[u] = fmaf(sums[(sec * 16 + wave * 4 + u) * 64 + lane], section_sign(sec * kSection), y[u]);
  float probe = 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u) probe = fmaf(y[u], 0.f, probe);
  if (__syncthreads_or(!(probe == 0.f))) {
    const f32x16 acc = fp32_block(o, m0, n0);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (wave == q && !__builtin_isfinite(y[u])) y[u] = acc[4 * q + u];
  }
  if (row < o.ntot) store_quad(o, f32x4{y[0], y[1], y[2], y[3]}, row, n0 + 8 * wave + 4 * lh);
}
__device__ __forceinline__ void update_few(const Operands& o) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int l32 = lane & 31, lh = lane >> 5;
  const int nct = o.N >> 5, ntiles = ((o.ntot + 31) >> 5) * nct, nk = o.nseg * o.d / 16;
  for (int tile = blockIdx.x * 4 + wave; tile < ntiles; tile += 4 * gridDim.x) {
    const int m0 = (tile / nct) * 32, n0 = (tile % nct) * 32, row = m0 + l32;
    const size_t aoff = (size_t)min(row, o.ntot - 1) * o.d + 8 * lh;
    const u32x4* wp = o.Ws + (size_t)lh * o.N + n0 + l32;
    f32x16 total = zero16(), acc = zero16();
    FewChunk s0, s1, s2, s3;
    few_fetch(o, s0, 0, aoff, wp);
    few_fetch(o, s1, min(1, nk - 1), aoff, wp);
    few_fetch(o, s2, min(2, nk - 1), aoff, wp);
    for (int c = 0; c < nk; c += kSection) {
      few_step<0>(o, total, acc, s0, s3, c, nk, aoff, wp);
      few_step<1>(o, total, acc, s1, s0, c + 1, nk, aoff, wp);
      few_step<2>(o, total, acc, s2, s1, c + 2, nk, aoff, wp);
      few_step<3>(o, total, acc, s3, s2, c + 3, nk, aoff, wp);
    }
    if (__any(!(finite_probe(total, 0.f) == 0.f))) total = mended(total, fp32_block(o, m0, n0));
    store_block(o, total, row, n0, lh);
  }
}

// ---------------------------------------------------------------------------
// tiles of 128 rows x 32 NB columns: four waves of 32 rows each
// ---------------------------------------------------------------------------
// Two workgroups per CU (two waves per SIMD), which do not wait for each other.  W goes through LDS, 24 KB a step
// (8 / NB chunks), double-buffered; a wave loads its own rows straight into registers, one or two steps ahead.  With
// NB = 4 a wave has 48 products of 32 cycles per step and reads 24 KB of W from LDS: 64 of the 128 bytes that LDS
// gives per cycle, so the matrix cores are the bound.  128 columns are the most that totals and sections leave
// registers for at two waves per SIMD.
// Order of a chunk's instructions: the reads of the third piece of W, then two vector instructions (of the splitting)
// behind every product, and the next piece's reads behind the first products of a piece.
template <int NB>
__device__ __forceinline__ void interleave() {
  __builtin_amdgcn_sched_group_barrier(0x100, NB, 0);                // LDS reads
#pragma unroll
  for (int p = 2; p >= 0; --p)
#pragma unroll
    for (int k = 0; k < (3 - p) * NB; ++k) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);             // product
      if (p > 0 && k < NB) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 8 / NB, 0);        // vector instructions
    }
}
template <int NB>
__global__ __launch_bounds__(256, 2) void update_split_kernel(Operands o, const int* __restrict__ node_off, int C, int few,
                                                              const int* __restrict__ status) {
  if (status[0] != 0) return;
  constexpr int BN = 32 * NB, CH = 8 / NB, U = 3 * CH * BN / 256;
  constexpr int kRound = CH > kSection ? CH : kSection;          // chunks of a round of the loop: whole steps, whole sections
  constexpr int kAhead = 4;                                      // chunks that rows are requested ahead of their splitting
  __shared__ u32x4 Wl[2][6 * CH * BN];
  o.ntot = node_off[C];
  if (few_tiles(o.ntot, o.N, gridDim.x) && (o.nseg * o.d + 16 * kSection - 1) / (16 * kSection) * 4096 <= (int)sizeof(Wl)) {
    update_fewer(o, reinterpret_cast<float*>(&Wl[0][0]));
    return;
  }
  if (few_tiles(o.ntot, o.N, few)) {
    update_few(o);
    return;
  }
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int l32 = lane & 31, lh = lane >> 5;
  const int nct = o.N / BN, ntiles = ((o.ntot + 127) >> 7) * nct;
  const int nk = o.nseg * o.d / 16, nstep = (nk + CH - 1) / CH;
  // a contiguous part of the tiles per XCD: the column tiles of a row tile read the same rows
  const int xcd = blockIdx.x & 7, per = gridDim.x >> 3;
  const int t1 = (int)((long long)ntiles * (xcd + 1) / 8);
  for (int tile = (int)((long long)ntiles * xcd / 8) + (blockIdx.x >> 3); tile < t1; tile += per) {
    const int m0 = (tile / nct) * 128 + wave * 32, n0 = (tile % nct) * BN, row = m0 + l32;
    const size_t aoff = (size_t)min(row, o.ntot - 1) * o.d + 8 * lh;
    auto fetch_a = [&](f32x4 (&x)[2], int c) {
      const float* a = chunk_base(o, c) + aoff;
      x[0] = *reinterpret_cast<const f32x4*>(a);
      x[1] = *reinterpret_cast<const f32x4*>(a + 4);
    };
    // half a step's W at a time
    auto fetch_w = [&](u32x4 (&w)[U], int s, int half) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = t + 256 * (u + half * U), r = min(s * CH * 6 + i / BN, nk * 6 - 1);
        w[u] = o.Ws[(size_t)r * o.N + n0 + i % BN];
      }
    };
    auto stash_w = [&](const u32x4 (&w)[U], int buf, int half) {
#pragma unroll
      for (int u = 0; u < U; ++u) Wl[buf][t + 256 * (u + half * U)] = w[u];
    };
    f32x16 total[NB], acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) total[j] = acc[j] = zero16();
    u32x4 w[U];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      fetch_w(w, 0, half);
      stash_w(w, 0, half);
    }
    f32x4 x[kAhead][2];                                  // rows of chunks c + 1 .. c + kAhead, chunk c in place c % kAhead
#pragma unroll
    for (int i = 0; i < kAhead; ++i) fetch_a(x[i], i);
    Pieces a = split8(x[0][0], x[0][1]);
    fetch_a(x[0], kAhead);
    __syncthreads();
    // full: every chunk of the round exists
    auto round = [&](int c0, auto full) {
#pragma unroll
      for (int i = 0; i < kRound; ++i) {
        const int c = c0 + i, s = c / CH, buf = s & 1;
        if (!full.value && i % CH == 0 && c >= nk) break;        // no such step
        if (i % CH == 0) fetch_w(w, s + 1, 0);
        if (i % CH == CH / 2) {                          // the other buffer was last read a step ago, before that step's barrier
          stash_w(w, buf ^ 1, 0);
          fetch_w(w, s + 1, 1);
        }
        __builtin_amdgcn_sched_barrier(0);               // the requests stay ahead of the products
        if (full.value || c < nk) {
          const u32x4* wl = &Wl[buf][(i % CH * 6 + lh) * BN + l32];
          u32x4 b[3][NB];
#pragma unroll
          for (int p = 2; p >= 0; --p) {
#pragma unroll
            for (int j = 0; j < NB; ++j) b[p][j] = wl[p * 2 * BN + j * 32];
#pragma unroll
            for (int q = 2 - p; q >= 0; --q)
#pragma unroll
              for (int j = 0; j < NB; ++j)
                acc[j] = product(b[p][j], a.p[q], i % kSection == 0 && p == 2 ? zero16() : acc[j]);
          }
          // the next chunk is split between this one's products
          a = split8(x[(i + 1) % kAhead][0], x[(i + 1) % kAhead][1]);
          if (full.value) interleave<NB>();
          __builtin_amdgcn_sched_barrier(0);
          fetch_a(x[(i + 1) % kAhead], c + 1 + kAhead);
          if (i % kSection == kSection - 1 || (!full.value && c == nk - 1))
#pragma unroll
            for (int j = 0; j < NB; ++j) add_section(total[j], acc[j], section_sign(c));
        }
        if (i % CH == CH - 1) {
          stash_w(w, buf ^ 1, 1);
          __syncthreads();
        }
      }
    };
    int c0 = 0;
    for (; c0 + kRound <= nk; c0 += kRound) round(c0, std::true_type{});
    if (c0 < nk) round(c0, std::false_type{});
    float probe = 0.f;
#pragma unroll
    for (int j = 0; j < NB; ++j) probe = finite_probe(total[j], probe);
    if (__any(!(probe == 0.f))) {
      if (m0 < o.ntot)
#pragma unroll
        for (int j = 0; j < NB; ++j) store_block(o, mended(total[j], fp32_block(o, m0, n0 + 32 * j)), row, n0 + 32 * j, lh);
    } else {
#pragma unroll
      for (int j = 0; j < NB; ++j) store_block(o, total[j], row, n0 + 32 * j, lh);
    }
  }
}

// ---------------------------------------------------------------------------
// weight gradients: C [M, N] = sum over rows r of [A0 | A1 | A2][r][:]^T B[r][:], M = nseg * d
// ---------------------------------------------------------------------------
// One workgroup = one 128 x 128 tile of C over one slab of rows, four waves of 64 x 64; two workgroups per CU.  The
// contraction index is the batch row: a thread loads two columns of eight rows, splits them and writes the pieces to LDS
// the way the products read them (eight rows of a column = 16 bytes), 16 rows a step, double-buffered; rows are requested two
// steps ahead.  Sections are 64 rows here; the pieces of B are negated in every other one.  Per step a wave has 24 products
// (768 cycles) and 110 vector instructions of splitting and adding sections, which other waves' products cover.
// A slab of few rows is one broken section, so every other slab begins with the negated sign: what is dropped cancels between
// them (160 rows in ten slabs, gradients of H = 256: 1.9e-7 off without, 1.42e-7 with).
// The column sums of B (bias gradients) ride along in the first row of tiles, in 64 bits: slabs are sixteen rows or more,
// which sums in fp32 would show (1.45e-7 against 1.17e-7; the pass takes the same time).  Partial results of the slabs are summed in
// a fixed order afterwards, so a pass is bit-reproducible.
// Up to kDirectRows rows a slab (a chunk) the rows are dealt as evenly as they go and the products are fp32 instructions on operands
// straight from memory: most of a chunk would be zeros, and with a row or two per slab a sum in 64 bits over the slabs follows,
// which six roundings per product would spoil (gradient of W2, 60 samples, H = 128: 5.0e-8 off in pieces, 2.8e-8 now).
constexpr int kDirectRows = 16;
constexpr int kWgT = 128;
struct WgradOperands {
  const float *A0, *A1, *A2, *B;
  float* part;
  long long part_stride;
  int d, nseg, N, ldb, S;
};
struct RowPairs {
  float2 r[8];         // two columns of eight rows
};
__global__ __launch_bounds__(256, 2) void wgrad_split_kernel(const WgradOperands o, const int* __restrict__ nrows,
                                                             const int* __restrict__ status) {
  if (status[0] != 0) return;
  __shared__ u32x4 L[2][6 * 2 * kWgT];         // [buffer][piece, half][128 columns of A, 128 of B]
  const int M = o.nseg * o.d, N = o.N;
  const int tiles_n = (N + kWgT - 1) / kWgT, tiles_m = (M + kWgT - 1) / kWgT, ntile = tiles_m * tiles_n;
  // Workgroups go round-robin to the eight XCDs: workgroup b becomes work item (b % 8) * (grid / 8) + b / 8, so that the
  // tiles of one slab, which read the same rows, run on one XCD (the grid is ntile * S with S a multiple of 8).
  const int item = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int tile = item % ntile, slab = item / ntile;
  const int m0 = (tile / tiles_n) * kWgT, n0 = (tile % tiles_n) * kWgT;
  const int rows = nrows[0];
  const int even = (rows + o.S - 1) / o.S;
  const bool direct = even <= kDirectRows;
  const int per = direct ? even : (even + 15) & ~15;
  const int r0 = (int)min((long long)slab * per, (long long)rows), r1 = min(r0 + per, rows);
  const int nchunk = direct ? 0 : (r1 - r0 + 15) >> 4;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, lh = lane >> 5;

  // loader: columns 2 cp and 2 cp + 1 of the 256 in LDS, rows 8 half .. + 7 of a chunk
  const int half = t >> 7, cp = t & 127;
  const bool is_b = cp >= kWgT / 2;
  const int col = is_b ? n0 + 2 * cp - kWgT : m0 + 2 * cp;
  const bool col_ok = col < (is_b ? N : M);            // both are even
  const int seg = is_b || !col_ok ? 0 : col / o.d;
  const float* src = is_b ? o.B : (seg == 0 ? o.A0 : (seg == 1 ? o.A1 : o.A2));
  const size_t ld = is_b ? o.ldb : o.d;
  src += col_ok ? col - seg * o.d : 0;
  const bool whole = m0 + kWgT <= M && n0 + kWgT <= N;
  auto fetch = [&](RowPairs& x, int c) {
    const int rb = r0 + c * 16 + 8 * half;
#pragma unroll
    for (int k = 0; k < 8; ++k) x.r[k] = *reinterpret_cast<const float2*>(src + (size_t)min(rb + k, r1 - 1) * ld);
  };
  double bsum[2] = {0.0, 0.0};
  const bool flip = slab & 1;
  // odd: the chunk belongs to an odd section
  auto stash = [&](RowPairs& x, int c, auto odd) {
    if (!whole || r0 + c * 16 + 16 > r1) {
      const int rb = r0 + c * 16 + 8 * half;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const bool keep = col_ok && rb + k < r1;
        x.r[k].x = keep ? x.r[k].x : 0.f;
        x.r[k].y = keep ? x.r[k].y : 0.f;
      }
    }
    if (m0 == 0 && is_b) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        bsum[0] += (double)x.r[k].x;
        bsum[1] += (double)x.r[k].y;
      }
    }
    u32x4* dst = &L[c & 1][half * 2 * kWgT + 2 * cp];
    if ((odd.value != 0) != flip && is_b) {
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        x.r[k].x = -x.r[k].x;
        x.r[k].y = -x.r[k].y;
      }
    }
    const Pieces p0 = split8(f32x4{x.r[0].x, x.r[1].x, x.r[2].x, x.r[3].x}, f32x4{x.r[4].x, x.r[5].x, x.r[6].x, x.r[7].x});
    const Pieces p1 = split8(f32x4{x.r[0].y, x.r[1].y, x.r[2].y, x.r[3].y}, f32x4{x.r[4].y, x.r[5].y, x.r[6].y, x.r[7].y});
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      dst[p * 4 * kWgT] = p0.p[p];
      dst[p * 4 * kWgT + 1] = p1.p[p];
    }
  };
  f32x16 total[2][2], acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) total[i][j] = acc[i][j] = zero16();
  // chunk c multiplies; chunk c + 1 goes from x to LDS; chunk c + 3 is requested into x
  auto step = [&](int c, RowPairs& x, auto in_section, auto odd, auto next_odd) {
    const u32x4* la = &L[c & 1][lh * 2 * kWgT + wm * 64 + l32];
    const u32x4* lb = &L[c & 1][lh * 2 * kWgT + kWgT + wn * 64 + l32];
    u32x4 a[3][2], b[2];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int i = 0; i < 2; ++i) a[p][i] = la[p * 4 * kWgT + 32 * i];
    if (c + 1 < nchunk) stash(x, c + 1, next_odd);
    if (c + 3 < nchunk) fetch(x, c + 3);
#pragma unroll
    for (int p = 2; p >= 0; --p) {
#pragma unroll
      for (int j = 0; j < 2; ++j) b[j] = lb[p * 4 * kWgT + 32 * j];
#pragma unroll
      for (int q = 2 - p; q >= 0; --q)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = product(b[j], a[q][i], in_section.value == 0 && p == 2 ? zero16() : acc[i][j]);
    }
    if (in_section.value == kSection - 1 || c == nchunk - 1)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) add_section(total[i][j], acc[i][j], (odd.value != 0) != flip ? -1.f : 1.f);
    __syncthreads();
  };
#define DC_INT(v_) std::integral_constant<int, v_>{}
  if (nchunk > 0) {
    RowPairs x0, x1;
    fetch(x0, 0);
    stash(x0, 0, DC_INT(0));
    if (nchunk > 1) fetch(x0, 1);
    if (nchunk > 2) fetch(x1, 2);
    __syncthreads();
    for (int c = 0; c < nchunk; c += 8) {
      step(c, x0, DC_INT(0), DC_INT(0), DC_INT(0));
      if (c + 1 < nchunk) step(c + 1, x1, DC_INT(1), DC_INT(0), DC_INT(0));
      if (c + 2 < nchunk) step(c + 2, x0, DC_INT(2), DC_INT(0), DC_INT(0));
      if (c + 3 < nchunk) step(c + 3, x1, DC_INT(3), DC_INT(0), DC_INT(1));
      if (c + 4 < nchunk) step(c + 4, x0, DC_INT(0), DC_INT(1), DC_INT(1));
      if (c + 5 < nchunk) step(c + 5, x1, DC_INT(1), DC_INT(1), DC_INT(1));
      if (c + 6 < nchunk) step(c + 6, x0, DC_INT(2), DC_INT(1), DC_INT(1));
      if (c + 7 < nchunk) step(c + 7, x1, DC_INT(3), DC_INT(1), DC_INT(0));
    }
  }
#undef DC_INT
  float probe = 0.f;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) probe = finite_probe(total[i][j], probe);
  const bool redo = __any(!(probe == 0.f));
  if (direct && r0 < r1) {
    // columns of A and B of the wave's two blocks each; pair k of rows, lanes 32-63 the second row of it
    float x[2][kDirectRows / 2], y[2][kDirectRows / 2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int mc = min(m0 + wm * 64 + 32 * i + l32, M - 1), mseg = mc / o.d;
      const float* am = (mseg == 0 ? o.A0 : (mseg == 1 ? o.A1 : o.A2)) + (mc - mseg * o.d);
      const float* bn = o.B + min(n0 + wn * 64 + 32 * i + l32, N - 1);
#pragma unroll
      for (int k = 0; k < kDirectRows / 2; ++k) {
        const int r = r0 + 2 * k + lh, rr = min(r, r1 - 1);
        const float a = am[(size_t)rr * o.d], b = bn[(size_t)rr * o.ldb];
        x[i][k] = r < r1 ? a : 0.f;
        y[i][k] = r < r1 ? b : 0.f;
      }
    }
#pragma unroll
    for (int k = 0; k < kDirectRows / 2; ++k)
      if (2 * k < r1 - r0)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) total[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(y[j][k], x[i][k], total[i][j], 0, 0, 0);
    if (m0 == 0 && is_b) {
      RowPairs b;
      fetch(b, 0);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const bool keep = r0 + 8 * half + k < r1;
        bsum[0] += keep ? (double)b.r[k].x : 0.0;
        bsum[1] += keep ? (double)b.r[k].y : 0.0;
      }
    }
  }
  float* P = o.part + (size_t)slab * (size_t)o.part_stride;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = m0 + wm * 64 + 32 * i + l32;
    const int mc = min(m, M - 1), mseg = mc / o.d;
    const float* am = (mseg == 0 ? o.A0 : (mseg == 1 ? o.A1 : o.A2)) + (mc - mseg * o.d);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int nb = n0 + wn * 64 + 32 * j;
      if (redo) {                                      // in fp32 instructions, straight from memory
        const float* bn = o.B + min(nb + l32, N - 1);
        f32x16 fp32 = zero16();
        for (int r = r0; r < r1; r += 2) {
          const int rr = min(r + lh, r1 - 1);
          const float x = r + lh < r1 ? am[(size_t)rr * o.d] : 0.f, y = r + lh < r1 ? bn[(size_t)rr * o.ldb] : 0.f;
          fp32 = __builtin_amdgcn_mfma_f32_32x32x2f32(y, x, fp32, 0, 0, 0);
        }
        total[i][j] = mended(total[i][j], fp32);
      }
      if (m < M) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int n = nb + 8 * q + 4 * lh;
          if (n < N)                                   // N is a multiple of 4
            *reinterpret_cast<f32x4*>(P + (size_t)m * N + n) =
                f32x4{total[i][j][4 * q], total[i][j][4 * q + 1], total[i][j][4 * q + 2], total[i][j][4 * q + 3]};
        }
      }
    }
  }
  if (m0 == 0) {                                       // the same for the whole workgroup
    double* sum = reinterpret_cast<double*>(&L[0][0]); // [2][128]
    __syncthreads();
    if (is_b) {
      sum[half * kWgT + 2 * cp - kWgT] = bsum[0];
      sum[half * kWgT + 2 * cp - kWgT + 1] = bsum[1];
    }
    __syncthreads();
    if (t < kWgT && n0 + t < N) P[(size_t)M * N + n0 + t] = (float)(sum[t] + sum[kWgT + t]);
  }
}

}  // namespace

void launch_wgrad_split(const float* A0, const float* A1, const float* A2, int d, int nseg, const float* B, int ldb, int N,
                        const int* nrows, float* part, long long part_stride, int S, const int* status, hipStream_t s) {
  const WgradOperands o{A0, A1, A2, B, part, part_stride, d, nseg, N, ldb, S};
  const int ntile = wgrad_split_tiles(nseg * d, N);
  hipLaunchKernelGGL(wgrad_split_kernel, dim3(ntile * S), dim3(256), 0, s, o, nrows, status);
}
int wgrad_split_tiles(int M, int N) { return ((M + kWgT - 1) / kWgT) * ((N + kWgT - 1) / kWgT); }

void launch_pack_split(const SplitJobs& jobs, int n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(pack_split_kernel, dim3(64, n), dim3(256), 0, s, jobs);
}

void launch_update_split(const GnnArgs& a, const float* A0, const float* A1, const float* A2, int d, int nseg, const float* Wf,
                         const unsigned short* Ws, const float* bias, float* out, hipStream_t s, bool transposed) {
  const Operands o{A0, A1, A2, reinterpret_cast<const u32x4*>(Ws), Wf, bias, out, d, nseg, a.H, 0,
                   transposed ? 1 : a.H, transposed ? nseg * d : 1};
  const dim3 grid((a.n_cu + 3) / 4 * 8), block(256);     // a multiple of eight
  const int few = 4 * a.n_cu;
  if (a.H % 128 == 0) hipLaunchKernelGGL(update_split_kernel<4>, grid, block, 0, s, o, a.node_off, a.n_cand, few, a.status);
  else if (a.H % 64 == 0) hipLaunchKernelGGL(update_split_kernel<2>, grid, block, 0, s, o, a.node_off, a.n_cand, few, a.status);
  else hipLaunchKernelGGL(update_split_kernel<1>, grid, block, 0, s, o, a.node_off, a.n_cand, few, a.status);
}

}  // namespace dc
