// Graph contraction of fusion candidates (gfx950).
//
// A candidate is a base training DAG plus one label per node; nodes with equal
// labels form one fused op or one fused gradient tensor (strategy space of
// Sec. 3.2).  The fused op is the subgraph of its original ops (Sec. 3.3), so the
// candidate module is the quotient graph: dependencies inside a group vanish,
// those that cross groups stay, parallel ones collapse (0/1 adjacency,
// Sec. 3.3.1).  Node features are summed per group (Sec. 2.3: the size of a fused
// tensor is the sum of its members' sizes).
//
// One workgroup contracts one candidate entirely in LDS (or, for base graphs
// that do not fit, in what LDS takes of its working arrays and a per-workgroup
// slab of global memory for the others).  Results go to per-candidate scratch slots; after a scan of the
// contracted sizes over the batch a second kernel places them block-diagonally
// and reduces the features.
//
// Output is canonical, hence unique: groups are numbered by ascending smallest
// member index and every neighbour list is ascending.
#include <limits.h>

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace dc {
namespace {

constexpr int kTinyRow = 4;     // lists up to this length are sorted where they are met, by one thread in registers,
constexpr int kSmallRow = 16;   // up to this length by one thread once all such are known, up to twice this by one thread where
                                // there are many, up to 64 by a wave
constexpr int kBmWaves = 2;     // waves that can always sort neighbour lists of more than 64 entries, through a bitmap each
constexpr unsigned short kSelf = 0xFFFF;

typedef unsigned short u16;
typedef unsigned long long u64;

// Working arrays of a candidate that fits LDS (byte offsets, the same on host and device).  nd = 2: successors and
// predecessors as one array of 2 G rows, nd = 1: one after the other.
//   ids:    u16 NID[N]: labels, then contracted ids | bitmaps, row numbers set aside, then masks (nd = 2: in the ids' place)
//   first:  MS[N + 1] group ends, int FIRST[N] (then u16 MEM[N], LST), u64 HM / u16 HP: heads and their ranks
//   later:  OFF[nd N + 1] row ends, u16 RAW[nd E] neighbours by row, then what sort_unique_32 may read
struct Slab {
  int nid, lst2, longest2, bm, mask, pre, ms, first, hm, hp, off, raw, nd, total;
  int bm_more, bm_waves;          // bitmaps of the waves behind the first kBmWaves, and how many waves have one
};
__host__ __device__ inline int align16(int x) { return (x + 15) & ~15; }
// Lists sorted where they are met: with one direction after the other LDS is short, and fewer numbers are set aside
__host__ __device__ inline int first_pass(int nd) { return nd == 2 ? kTinyRow : 2 * kTinyRow; }
__host__ __device__ inline Slab slab_layout_nd(int N, int E, int nd) {
  constexpr int os = 2;                    // counters and ends of rows are 16-bit
  Slab s;
  s.total = INT_MAX;
  if ((long long)nd * E > 65535) return s;
  const int rows = nd * N, slots = nd * E, w = (slots + 63) / 64 + 1, hw = (N + 63) / 64 + 1;
  s.nd = nd;
  s.nid = 0;
  const int ids = align16(2 * (N + 2));
  const int bm = align16(4 * kBmWaves * ((N + 31) / 32 + 1)), mask = align16(8 * w) + align16(4 * w);
  const int lst = align16(os * (slots / (first_pass(nd) + 1) + 2));
  const int longest = align16(os * (slots / (kSmallRow + 1) + 2));
  const int aux = bm + (mask > lst + longest ? mask : lst + longest);
  const int x = nd == 2 && aux > ids ? aux : ids;
  int o = x;
  s.ms = o;    o = align16(o + os * (N + 2));
  s.first = o; o = align16(o + 4 * N + 4 * os);
  s.hm = o;    o = align16(o + 8 * hw);
  s.hp = o;    o = align16(o + 2 * hw);
  s.total = o;
  o = x;
  s.off = o;   o = align16(o + os * (rows + 2));
  s.raw = o;   o = align16(o + 2 * (slots + kSmallRow));
  s.bm = nd == 2 ? 0 : o;                  // one after the other: the ids are needed again
  s.lst2 = s.mask = s.bm + bm;
  s.longest2 = s.lst2 + lst;
  s.pre = s.mask + align16(8 * w);
  if (nd == 1) o += aux;
  if (o > s.total) s.total = o;
  s.bm_more = s.total;
  s.bm_waves = kBmWaves;
  return s;
}
// Both directions at once, in half the phases, where that fits.
__host__ __device__ inline Slab slab_layout(int N, int E, int lds) {
  Slab s = slab_layout_nd(N, E, 2);
  if (s.total > lds) s = slab_layout_nd(N, E, 1);
  s.bm_more = s.total;                     // the LDS that is left, up to a bitmap for each of sixteen waves
  const int more = (lds - s.total) / (4 * ((N + 31) / 32 + 1));
  s.bm_waves = kBmWaves + (more < 16 - kBmWaves ? more : 16 - kBmWaves);
  return s;
}
__host__ __device__ inline int slab_need(int N, int E) { return slab_layout_nd(N, E, 1).total; }

// The working arrays of a candidate that does not fit LDS: one direction after the other, counters of 16 bits up to 65535 edges
// and of 32 beyond.  An array goes to LDS while there is room, in the order in which they are asked for, which is how
// much their accesses are dependent on each other; sizes that are only known as the candidate is contracted (groups, edges
// between groups) are asked for as they are.  One candidate of 21 k nodes and 34 k edges 660 us with all arrays in global memory,
// 213 us; of 65 k nodes and 107 k edges 2.03 and 1.18 ms; 256 of 700 nodes and 66 k edges 4.06 and 0.31 ms.
template <typename T>
struct Split {                             // an array whose first `cap` entries (a multiple of sixteen) lie apart from the others
  T *near, *far;
  int cap;
  __device__ __forceinline__ T* of(int i) const { return i < cap ? near : far; }
  __device__ __forceinline__ T& operator[](int i) const { return of(i)[i]; }
};
template <typename T>
__device__ __forceinline__ T* part_of(const Split<T>& a, int i) { return a.of(i); }
template <typename T>
__device__ __forceinline__ T* part_of(T* a, int) { return a; }
struct Places {
  char *lds, *lds_end, *slab;
  __device__ __forceinline__ char* take(size_t bytes, size_t spare = 0) {      // spare: of the LDS, for a later array
    bytes = (bytes + 15) & ~(size_t)15;
    char* p;
    if (bytes + spare <= (size_t)(lds_end - lds)) {
      p = lds;
      lds += bytes;
    } else {
      p = slab;
      slab += bytes;
    }
    return p;
  }
  // n entries, as many of them in LDS as there is room for
  template <typename T>
  __device__ __forceinline__ Split<T> take_split(int n) {
    const int cap = min((n + 15) & ~15, (int)((lds_end - lds) / sizeof(T)) & ~15);
    Split<T> s{reinterpret_cast<T*>(lds), reinterpret_cast<T*>(slab) - cap, cap};
    lds += cap * sizeof(T);
    if (n > cap) slab += ((size_t)(n - cap) * sizeof(T) + 15) & ~(size_t)15;
    return s;
  }
};
inline size_t slab_bytes(int N, int E) {                  // of Places without any LDS
  const size_t n = N, e = E, mask = 12 * ((e + 63) / 64 + 1), lst = 2 * (e / (2 * kTinyRow + 1) + e / (kSmallRow + 1) + 4);
  const size_t relabel = 10 * ((n + 63) / 64 + 1) + 4 * n + 8 + 2 * (n + 2);
  const size_t lists = 4 * (n + 2) + 2 * (e + kSmallRow) + (mask > lst ? mask : lst) + 64 * ((n + 31) / 32);
  return 2 * (n + 2) + (relabel > lists ? relabel : lists) + 16 * 16;
}

// Classes of base graphs by working set (one direction after the other): four, two and one workgroup per CU, which its 16
// waves of some 110 registers allow; a workgroup takes its share of the LDS.  1024 candidates of 1.6 k nodes: 131 us with
// sixteen waves each, 45 us with four; 4096 of 6.6 k nodes: 762 us with eight waves, 584 with sixteen.
constexpr int kStatic = 256;               // static LDS of the kernel
struct SizeClass {
  int most, lds, threads;
};
__host__ __device__ inline SizeClass size_class_of(int k, int lds_limit) {
  const int lds = k == 2 ? lds_limit : (40960 << k) - kStatic, share = lds < lds_limit ? lds : lds_limit;
  return {k == 2 ? share : share / 2, share, 256 << k};
}

// Short lists (up to 16 entries) are sorted by one thread each, in registers, with a
// fixed compare-exchange network (Batcher's odd-even merge sort): no dependent chain
// through memory, and the same instruction stream for every lane.  Unused places hold
// kSelf (0xFFFF), which sorts to the end.
template <int NN, typename T>
__device__ __forceinline__ void compare_exchange(T (&v)[NN], int i, int j) {
  const T lo = __builtin_elementwise_min(v[i], v[j]), hi = __builtin_elementwise_max(v[i], v[j]);
  v[i] = lo;
  v[j] = hi;
}
template <int NN, typename T>
__device__ __forceinline__ void sort_network(T (&v)[NN]) {
#pragma unroll
  for (int p = 1; p < NN; p <<= 1)
#pragma unroll
    for (int k = p; k >= 1; k >>= 1)
#pragma unroll
      for (int j = k % p; j + k < NN; j += 2 * k)
#pragma unroll
        for (int i = 0; i < k; ++i)
          if (i + j + k < NN && (i + j) / (2 * p) == (i + j + k) / (2 * p)) compare_exchange<NN>(v, i + j, i + j + k);
}

// Sorts a[0..n) ascending, n <= NN; kSelf in the place of a repeat.  The reads are unconditional (a[0] is readable with
// n = 0 too): behind a condition each would wait for the one before it.
template <int NN>
__device__ __forceinline__ void sort_unique_small(u16* a, int n) {
  unsigned v[NN];
#pragma unroll
  for (int k = 0; k < NN; ++k) v[k] = a[min(k, max(n - 1, 0))];
#pragma unroll
  for (int k = 0; k < NN; ++k) v[k] = k < n ? v[k] : (unsigned)kSelf;
  sort_network<NN>(v);
#pragma unroll
  for (int k = 0; k < NN; ++k)
    if (k < n) a[k] = (k > 0 && v[k] == v[k - 1]) ? kSelf : (u16)v[k];
}

// Same for 17 to 32 entries, two to a register (a register each leaves the kernel none to work with): entries i and i + 16 are
// sorted side by side, and what is left is the merge of a bitonic sequence.  The 15 places behind a list's end are readable.
typedef u16 u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void sort_unique_32(u16* a, int n) {
  u16x2 w[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) w[k] = u16x2{a[k], a[k + 16]};
#pragma unroll
  for (int k = 0; k < 16; ++k) w[k].y = k + 16 < n ? w[k].y : kSelf;
  sort_network<16>(w);
#pragma unroll
  for (int k = 0; k < 8; ++k) {              // the upper half downwards
    const u16 y = w[k].y;
    w[k].y = w[15 - k].y;
    w[15 - k].y = y;
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const u16x2 s = w[k].yx;
    w[k] = u16x2{__builtin_elementwise_min(w[k], s).x, __builtin_elementwise_max(w[k], s).y};
  }
#pragma unroll
  for (int d = 8; d >= 1; d >>= 1)
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if ((k & d) == 0) compare_exchange<16>(w, k, k + d);
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    const u16 x = k < 16 ? w[k & 15].x : w[k & 15].y, before = k == 0 ? kSelf : (k <= 16 ? w[(k - 1) & 15].x : w[(k - 1) & 15].y);
    if (k < n) a[k] = k > 0 && x == before ? kSelf : x;
  }
}

// Same for up to 64 entries by a whole wave (lane i holds entry i): an entry's place is the number of smaller ones.
__device__ __forceinline__ void sort_wave(u16* a, int n, int lane) {
  const unsigned x = a[min(lane, n - 1)];
  const int key = lane < n ? (int)(x << 6) | lane : INT_MAX;
  int pos = 0;
  for (int j = 0; j < n; j += 4)             // four at a time: the compiler does not unroll a loop over lanes by itself
#pragma unroll
    for (int u = 0; u < 4; ++u) pos += __builtin_amdgcn_readlane(key, j + u) < key ? 1 : 0;
  if (lane < n) a[pos] = (u16)x;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  const u16 y = a[min(lane, n - 1)], before = a[max(min(lane, n - 1) - 1, 0)];
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  if (lane > 0 && lane < n && y == before) a[lane] = kSelf;
}

// A barrier for working arrays in LDS: results on their way to memory, which nobody reads here, are not waited for.
template <bool kLds>
__device__ __forceinline__ void block_sync() {
  if (kLds) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  } else {
    __syncthreads();
  }
}

// Counters: one more at place i, returns what was there.  16-bit ones lie in pairs (LDS has no 16-bit atomics); the
// arrays hold at most 65535 entries, so no counter carries into its neighbour.
__device__ __forceinline__ int count_one(u16* a, int i) {
  const int sh = (i & 1) * 16;
  return (int)((atomicAdd(reinterpret_cast<unsigned*>(a) + (i >> 1), 1u << sh) >> sh) & 0xFFFFu);
}
__device__ __forceinline__ int count_one(int* a, int i) { return atomicAdd(&a[i], 1); }
template <typename T>
__device__ __forceinline__ int count_one(const Split<T>& a, int i) { return count_one(a.of(i), i); }
// The 32-bit word w of an array: two counters of 16 bits or one of 32
template <typename A>
__device__ __forceinline__ int* word_of(const A& a, int w) {
  const int i = w * (int)(4 / sizeof(a[0]));
  return reinterpret_cast<int*>(part_of(a, i) + i);
}

// The sum over the waves in front of this one, and over all of them (`total`), of what each wave's last lane has in `inc`.
template <bool kLds>
__device__ __forceinline__ int wave_offsets(int inc, int& total, int* wsum) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, nw = blockDim.x >> 6;
  if (lane == 63) wsum[wave] = inc;
  block_sync<kLds>();
  const int x = wave_incl_scan(lane < nw ? wsum[lane & 15] : 0);
  total = __builtin_amdgcn_readlane(x, 63);
  return __builtin_amdgcn_readlane(x, wave) - __builtin_amdgcn_readlane(inc, 63);
}

// Exclusive scan in place; the entry behind the last is 0 before and may be anything after.  Returns the total.
template <bool kLds, typename A>
__device__ __forceinline__ int exscan16(const A& a, int n, int* wsum) {
  const int t = threadIdx.x, T = blockDim.x, nw = (n + 1) >> 1;
  const int K = ((nw + T - 1) / T) | 1;          // an odd run of words per thread: no two lanes of a half wave in one bank
  const int lo = min(t * K, nw), hi = min(lo + K, nw);
  int s = 0;
  for (int i = lo; i < hi; ++i) {
    const unsigned x = *word_of(a, i);
    s += (x & 0xFFFF) + (x >> 16);
  }
  const int inc = wave_incl_scan(s);
  int total;
  int run = wave_offsets<kLds>(inc, total, wsum) + inc - s;
  for (int i = lo; i < hi; ++i) {
    const unsigned x = *word_of(a, i);
    const int mid = run + (x & 0xFFFF);
    *word_of(a, i) = (int)((unsigned)run | ((unsigned)mid << 16));
    run = mid + (x >> 16);
  }
  block_sync<kLds>();
  return total;
}
template <bool kLds, typename A>
__device__ __forceinline__ int exscan(const A& a, int n, int* wsum) {
  if constexpr (sizeof(a[0]) == 2) return exscan16<kLds>(a, n, wsum);
  else return block_exscan_lines(a, a, n, wsum);
}

// pre[w] = bits set in front of word w of m, pre[nw] = all of them (returned); m[nw] = 0
template <bool kLds, typename Pre>
__device__ __forceinline__ int scan_bits(u64* m, Pre* pre, int nw, int* wsum) {
  const int t = threadIdx.x, T = blockDim.x;
  int carry = 0;
  for (int w0 = 0; w0 < nw; w0 += T) {
    const int w = w0 + t, pc = w < nw ? __popcll(m[w]) : 0;
    const int inc = wave_incl_scan(pc);
    int total;
    const int run = carry + wave_offsets<kLds>(inc, total, wsum) + inc - pc;
    if (w < nw) pre[w] = (Pre)run;
    carry += total;
    if (w0 + T < nw) block_sync<kLds>();         // wsum is written again
  }
  if (t == 0) {
    m[nw] = 0;
    pre[nw] = (Pre)carry;
  }
  block_sync<kLds>();
  return carry;
}
// Bit i of m: `set(i)`, i < n.  A wave takes kBatch words of 64 at a time.
template <int kBatch, typename Set>
__device__ __forceinline__ void fill_bits(u64* m, int n, Set set) {
  const int t = threadIdx.x, T = blockDim.x, lane = t & 63;
  for (int i0 = t & ~63; i0 < n; i0 += kBatch * T) {
    bool x[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) x[j] = set(min(i0 + j * T + lane, n - 1));
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int i = i0 + j * T;
      const u64 b = __ballot(x[j] && i + lane < n);
      if (lane == 0 && i < n) m[i >> 6] = b;
    }
  }
}
// Four neighbouring entries in one store; p is aligned to an entry only.
__device__ __forceinline__ void store4(int* p, int a, int b, int c, int d) {
  struct __attribute__((packed, aligned(4))) Quad { int x[4]; };
  *reinterpret_cast<Quad*>(p) = Quad{{a, b, c, d}};
}
// p[i] = value(i), i < n; a thread takes four neighbouring entries (a store costs a CU some 40 cycles whatever its width)
template <typename Value>
__device__ __forceinline__ void store_all(int* p, int n, Value value) {
  for (int i = 4 * threadIdx.x; i < n; i += 4 * blockDim.x) {
    if (i + 4 <= n) store4(p + i, value(i), value(i + 1), value(i + 2), value(i + 3));
    else for (int k = i; k < n; ++k) p[k] = value(k);
  }
}
template <typename Pre>
__device__ __forceinline__ int bits_before(const u64* m, const Pre* pre, int i) {
  return pre[i >> 6] + __popcll(m[i >> 6] & ((1ull << (i & 63)) - 1ull));
}

// Rows r < rows of `a`, row r ending at end[r], each ascending, kSelf in the place of a repeat.  Rows of up to `at_once`
// (four or eight) entries are sorted as they are met; the others are set aside, those of up to eight from the front of `lst`, of up to 16 from
// its back (`room` entries), so that the waves that sort them are full and take one network each.  More than 16
// entries: up to 32 from the front of `longest`, more from its back (`long_room` entries).  Those of up to 32 take a network too
// where there are more of them than waves (one candidate of 2.5 k nodes and 25 k edges: 225 us with a wave each, 96 us; 8192
// of 64 power-law graphs of up to 20 k nodes 2.01 -> 1.69 ms); the others `longer(r, begin, n)`, called by whole waves, all of
// them for up to 64 entries, the first `most` for more.  Member lists need no bitmap: one candidate with 50 groups of 100 of its 6.6 k nodes 328 us with two waves for them, 117 us
// with sixteen; one of 900 nodes with 33 k edges, nearly all lists longer than 64: 488 us with two bitmaps, 186 us with sixteen.
// cnt[0 .. 3] are 0.
template <bool kLds, typename End, typename Longer>
__device__ __forceinline__ void sort_rows(u16* a, const End& end, int rows, u16* lst, int room, int at_once, u16* longest,
                                          int long_room, int most, int* cnt, Longer longer) {
  const int t = threadIdx.x, T = blockDim.x, wave = t >> 6, lane = t & 63;
  auto begin = [&](int r) { return r ? (int)end[r - 1] : 0; };
  for (int r = t; r < rows; r += T) {
    const int s = begin(r), n = (int)end[r] - s;
    if (n <= kTinyRow) {
      if (n > 1) sort_unique_small<kTinyRow>(a + s, n);
    } else if (n <= at_once) {
      sort_unique_small<2 * kTinyRow>(a + s, n);
    } else if (n <= 2 * kTinyRow) {
      lst[atomicAdd(&cnt[0], 1)] = (u16)r;
    } else if (n <= kSmallRow) {
      lst[room - 1 - atomicAdd(&cnt[1], 1)] = (u16)r;
    } else if (n <= 2 * kSmallRow) {
      longest[atomicAdd(&cnt[2], 1)] = (u16)r;
    } else {
      longest[long_room - 1 - atomicAdd(&cnt[3], 1)] = (u16)r;
    }
  }
  block_sync<kLds>();
  const int all = T >> 6, n8 = cnt[0], n16 = cnt[1], n64 = cnt[2] > all ? 0 : cnt[2], n32 = cnt[2] - n64, nl = n64 + cnt[3];
  const int w8 = (n8 + 63) >> 6, w16 = (n16 + 63) >> 6, w32 = (n32 + 63) >> 6;
  for (int w = wave; w < w8 + w16 + w32; w += all) {
    if (w < w32) {                               // the longer network first
      const int i = w * 64 + lane;
      if (i < n32) {
        const int r = longest[i], s = begin(r);
        sort_unique_32(a + s, (int)end[r] - s);
      }
    } else if (w < w32 + w16) {
      const int i = (w - w32) * 64 + lane;
      if (i < n16) {
        const int r = lst[room - 1 - i], s = begin(r);
        sort_unique_small<kSmallRow>(a + s, (int)end[r] - s);
      }
    } else {
      const int i = (w - w32 - w16) * 64 + lane;
      if (i < n8) {
        const int r = lst[i], s = begin(r);
        sort_unique_small<2 * kTinyRow>(a + s, (int)end[r] - s);
      }
    }
  }
  // the last waves first: the first ones have the networks
  auto by_wave = [&](int i) { return (int)(i < n64 ? longest[i] : longest[long_room - 1 - (i - n64)]); };
  for (int i = all - 1 - wave; i < nl; i += all) {
    const int r = by_wave(i), s = begin(r), n = (int)end[r] - s;
    if (n <= 64 || most >= all) longer(r, s, n);
  }
  if (most < all && wave < most)
    for (int i = n64 + wave; i < nl; i += most) {
      const int r = by_wave(i), s = begin(r), n = (int)end[r] - s;
      if (n > 64) longer(r, s, n);
    }
  block_sync<kLds>();
}

// One candidate, working arrays in LDS (kLds, where `L` says) or in `places`.  Bound by the latency of its phases:
// about twenty, a barrier each, of a few dependent LDS accesses.  Edges are dealt to the threads as (source, target) pairs
// and counted, then placed, by group; those inside a group never enter a row.  What is left of the rows after sorting
// is found through a mask over their places, so that lists and row starts leave in order, whole lines at a time.
// One candidate of 6.5 k nodes and 10 k edges in 1.4 k groups: 58 us with a scan per direction over all members and lists
// gathered member by member, 36 us; 4096 of them 866 -> 584 us, 1000 of 6.5 k groups 224 -> 159 us; 8192 candidates of
// 64 graphs of up to 19 k nodes, the larger ones in global memory before, 4.9 -> 1.2 ms.
template <bool kLds, typename Off, int kBatch>
__device__ __forceinline__ void contract_one(const BaseGraphs& bg, int c, int b, int N, int E, char* base, const Slab& L, Places places,
                                             int lds_bytes, int coff, int eslot, const int* label, const ContractTmp& tmp,
                                             int* new_id_out, int* status, int* wsum) {
  const int t = threadIdx.x, T = blockDim.x, lane = t & 63, wave = t >> 6;
  // the array at byte `at` of the LDS layout, or the next place for `bytes`
  auto array = [&](int at, size_t bytes, size_t spare = 0) { return kLds ? base + at : places.take(bytes, spare); };
  u16* NID = reinterpret_cast<u16*>(array(L.nid, 2 * ((size_t)N + 2)));
  Places behind_ids = places;
  const int hw = ((N + 63) >> 6) + 1;
  u64* HM = reinterpret_cast<u64*>(array(L.hm, 8 * (size_t)hw));
  u16* HP = reinterpret_cast<u16*>(array(L.hp, 2 * (size_t)hw));
  int* FIRST = reinterpret_cast<int*>(array(L.first, 4 * (size_t)N + 8, 2 * (size_t)N));
  typedef typename std::conditional<kLds, u16*, Split<u16>>::type Groups;
  typedef typename std::conditional<kLds, Off*, Split<Off>>::type Ends;
  Groups MS;
  if constexpr (kLds) MS = reinterpret_cast<u16*>(base + L.ms);
  u16* MEM = reinterpret_cast<u16*>(FIRST);                       // once the ids are known
  u16* LST = reinterpret_cast<u16*>(reinterpret_cast<char*>(FIRST) + align16(2 * N));
  u16* LONGEST = LST + N / (kTinyRow + 1) + 1;
  int* cnt = wsum + 16;            // four words behind the scans' wave sums

  const int* lab = label + coff;
  int* nid_out = new_id_out + coff;
  const int nslot = coff + c;
  const unsigned* edge = bg.edge + bg.geo[b];

  // The lanes of a wave take nodes far from each other where they count or place by group: neighbours are mostly in one
  // group, and atomics on one word follow each other (edges lie in memory in such an order).  An odd distance: every
  // lane in a bank of its own.
  const int apart = ((N + 63) >> 6) | 1, spread = N > 0 ? apart << 6 : 0;
  auto node = [&](int i) { return i < spread ? (i & 63) * apart + (i >> 6) : N; };

  // ---- relabel: groups numbered by ascending smallest member -----------------
  int bad = 0;
  for (int v0 = t; v0 < N; v0 += kBatch * T) {
    int l[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) l[j] = lab[min(v0 + j * T, N - 1)];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int v = v0 + j * T;
      bad |= (l[j] < 0) | (l[j] >= N);
      if (v < N) {
        NID[v] = (u16)l[j];
        FIRST[v] = INT_MAX;
      }
    }
  }
  if constexpr (kLds)
    for (int i = t; i < (N + 2) / 2; i += T) *word_of(MS, i) = 0;
  if (t < 4) cnt[t] = 0;
  if (__syncthreads_or(bad)) {
    if (t == 0) {
      set_error(status, (int)DC_ERR_BAD_PARTITION);
      tmp.Gc[c] = 0;
      tmp.Ec[c] = 0;
    }
    return;
  }
  for (int i = t; i < spread; i += kBatch * T) {
    int l[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) l[j] = NID[min(node(i + j * T), N - 1)];
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      if (node(i + j * T) < N) atomicMin(&FIRST[l[j]], node(i + j * T));
  }
  block_sync<kLds>();
  fill_bits<kBatch>(HM, N, [&](int v) { return FIRST[NID[v]] == v; });
  block_sync<kLds>();
  const int G = scan_bits<kLds>(HM, HP, (N + 63) >> 6, wsum);
  if constexpr (!kLds) {
    MS = places.take_split<u16>(G + 2);
    for (int i = t; i < (G + 2) / 2; i += T) *word_of(MS, i) = 0;
    __syncthreads();
  }
  for (int i = t; i < spread; i += kBatch * T) {
    int g[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) g[j] = NID[min(node(i + j * T), N - 1)];
    // a place past the end is another thread's last one, which may hold its id already
#pragma unroll
    for (int j = 0; j < kBatch; ++j) g[j] = FIRST[node(i + j * T) < N ? g[j] : 0];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) g[j] = bits_before(HM, HP, node(i + j * T) < N ? g[j] : 0);
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int v = node(i + j * T);
      if (v < N) {
        NID[v] = (u16)g[j];
        count_one(MS, g[j]);
      }
    }
  }
  block_sync<kLds>();

  // ---- member lists: counting sort by group, then ascending inside a group ---------
  exscan<kLds>(MS, G, wsum);
  for (int i = t; i < spread; i += kBatch * T) {
    int g[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) g[j] = NID[min(node(i + j * T), N - 1)];
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      if (node(i + j * T) < N) g[j] = count_one(MS, g[j]);                 // MS[g] becomes the end of group g
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      if (node(i + j * T) < N) MEM[g[j]] = (u16)node(i + j * T);
  }
  block_sync<kLds>();
  sort_rows<kLds>(MEM, MS, G, LST, N / (kTinyRow + 1) + 1, kTinyRow, LONGEST, N / (kSmallRow + 1) + 1, T >> 6, cnt, [&](int g, int s, int n) {
    if (n <= 64) {
      sort_wave(MEM + s, n, lane);
      return;
    }
    // large groups: ordered compaction over all nodes
    int cnt = 0;
    for (int v0 = 0; v0 < N; v0 += 64) {
      const int v = v0 + lane;
      const bool f = v < N && NID[v] == g;
      const u64 m = __ballot(f);
      if (f) MEM[s + cnt + __popcll(m & ((1ull << lane) - 1ull))] = (u16)v;
      cnt += __popcll(m);
    }
  });
  store_all(nid_out, N, [&](int v) { return (int)NID[v]; });
  store_all(tmp.members + coff, N, [&](int i) { return (int)MEM[i]; });
  store_all(tmp.mstart + nslot, G + 1, [&](int g) { return g ? (int)MS[g - 1] : 0; });
  block_sync<kLds>();

  // ---- neighbour lists: successors are rows 0 .. G - 1, predecessors the next G (nd = 2), or one after the other ----------
  const int nd = kLds ? L.nd : 1;
  const int bm_words = kLds ? (N + 31) / 32 + 1 : (G + 31) / 32;
  if constexpr (!kLds) {
    // An edge costs 1.8 times as much with the ids in global memory, 3.3 times with the ends of rows there (atomics), so the
    // ids make room where that brings more than 36 % of the ends into LDS.
    auto in_lds = [&](const char* from) { return min((long long)G, (long long)((places.lds_end - from) / (long long)sizeof(Off))); };
    char* const all = places.lds_end - lds_bytes;
    if (reinterpret_cast<char*>(NID) == all && in_lds(all) - in_lds(behind_ids.lds) > (long long)G * 36 / 100) {
      u16* moved = reinterpret_cast<u16*>(behind_ids.slab);
      for (int v = t; v < N; v += T) moved[v] = NID[v];
      NID = moved;
      behind_ids.slab += (2 * ((size_t)N + 2) + 15) & ~(size_t)15;
      behind_ids.lds = all;
      __syncthreads();
    }
  }
  int Ec = 0;
  for (int dir = 0; dir < 2; dir += nd) {
    const int rows = nd * G;
    places = behind_ids;
    Ends OFF;
    if constexpr (kLds) OFF = reinterpret_cast<Off*>(base + L.off);
    else OFF = places.take_split<Off>(rows + 2);
    u16* RAW = nullptr;                                // its size is known after the counts
    for (int i = t; i < (int)(sizeof(Off) * (rows + 2)) / 4; i += T) *word_of(OFF, i) = 0;
    if (t < 4) cnt[t] = 0;
    block_sync<kLds>();
    // counts the edges between groups, or places them; the others and those past the end are left out
    auto each_edge = [&](auto place) {
      for (int e0 = t; e0 < E; e0 += kBatch * T) {
        unsigned x[kBatch];
        int gu[kBatch], gw[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) x[j] = edge[min(e0 + j * T, E - 1)];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
          gu[j] = NID[x[j] & 0xFFFF];
          gw[j] = NID[x[j] >> 16];
          if (e0 + j * T >= E) gw[j] = gu[j];
        }
        int po[kBatch], pi[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
          if (gu[j] != gw[j] && (nd == 2 || dir == 0)) po[j] = count_one(OFF, gu[j]);
          if (gu[j] != gw[j] && (nd == 2 || dir == 1)) pi[j] = count_one(OFF, (nd - 1) * G + gw[j]);
        }
        if (place.value) {
#pragma unroll
          for (int j = 0; j < kBatch; ++j) {
            if (gu[j] != gw[j] && (nd == 2 || dir == 0)) RAW[po[j]] = (u16)gw[j];
            if (gu[j] != gw[j] && (nd == 2 || dir == 1)) RAW[pi[j]] = (u16)gu[j];
          }
        }
      }
      block_sync<kLds>();
    };
    each_edge(std::false_type{});
    const int S = exscan<kLds>(OFF, rows, wsum);
    RAW = reinterpret_cast<u16*>(array(L.raw, 2 * ((size_t)S + kSmallRow)));
    each_edge(std::true_type{});
    // the rows set aside, and when they are sorted the mask over the places
    const size_t n_mask = ((size_t)S + 63) / 64 + 1, n_lst = (size_t)S / (first_pass(nd) + 1) + 1, n_longest = (size_t)S / (kSmallRow + 1) + 1;
    char* aux = array(L.lst2, n_mask * 12 > 2 * (n_lst + n_longest) ? n_mask * 12 : 2 * (n_lst + n_longest));
    u16* LST2 = reinterpret_cast<u16*>(aux);
    u16* LONGEST2 = kLds ? reinterpret_cast<u16*>(base + L.longest2) : LST2 + n_lst;
    u64* MASK = reinterpret_cast<u64*>(kLds ? base + L.mask : aux);
    int* PRE = reinterpret_cast<int*>(kLds ? base + L.pre : aux + 8 * n_mask);
    char* bitmaps = array(L.bm, 64 * (size_t)bm_words);
    unsigned* BM = reinterpret_cast<unsigned*>(kLds && wave >= kBmWaves ? base + L.bm_more + 4 * (wave - kBmWaves) * bm_words
                                                                       : bitmaps + 4 * wave * bm_words);
    bool clean = false;                                // the wave's bitmap is zero
    sort_rows<kLds>(RAW, OFF, rows, LST2, (int)n_lst, first_pass(nd), LONGEST2, (int)n_longest, kLds ? L.bm_waves : 16, cnt, [&](int, int s, int n) {
      if (n <= 64) {
        sort_wave(RAW + s, n, lane);
        return;
      }
      // mark neighbours in the wave's bitmap, then list the set bits
      if (!clean) {
        for (int i = lane; i < bm_words; i += 64) BM[i] = 0u;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        clean = true;
      }
      for (int i = lane; i < n; i += 64) {
        const u16 x = RAW[s + i];
        atomicOr(&BM[x >> 5], 1u << (x & 31));
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      int cnt = 0;
      for (int w0 = 0; w0 < (G + 31) / 32; w0 += 64) {
        const int w = w0 + lane;
        unsigned bits = (w < (G + 31) / 32) ? BM[w] : 0u;
        if (bits) BM[w] = 0u;
        const int pc = __popc(bits);
        const int inc = wave_incl_scan(pc);
        int o = s + cnt + inc - pc;
        while (bits) {
          RAW[o++] = (u16)((w << 5) + __ffs(bits) - 1);
          bits &= bits - 1;
        }
        cnt += __shfl(inc, 63, 64);
      }
      for (int i = cnt + lane; i < n; i += 64) RAW[s + i] = kSelf;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    });
    fill_bits<kBatch>(MASK, S, [&](int i) { return RAW[i] != kSelf; });
    block_sync<kLds>();
    const int kept = scan_bits<kLds>(MASK, PRE, (S + 63) >> 6, wsum);
    Ec = nd == 2 ? kept >> 1 : kept;                   // every kept edge is in one list of either kind
    int* col0 = (dir == 0 ? tmp.oc : tmp.ic) + eslot;
    int* col1 = tmp.ic + eslot;
    // four places per thread: mostly all of them are kept and leave together
    for (int s = 4 * t; s < S; s += 4 * T) {
      const u64 m = MASK[s >> 6];
      const unsigned four = (unsigned)(m >> (s & 63)) & 15u;
      int k = PRE[s >> 6] + __popcll(m & ((1ull << (s & 63)) - 1ull));
      if (four == 15u && (k >= Ec || k + 4 <= Ec)) {
        store4(k < Ec ? col0 + k : col1 + (k - Ec), RAW[s], RAW[s + 1], RAW[s + 2], RAW[s + 3]);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if ((four >> j) & 1u) {
            *(k < Ec ? col0 + k : col1 + (k - Ec)) = RAW[s + j];
            ++k;
          }
      }
    }
    auto row_start = [&](int r) { return r ? bits_before(MASK, PRE, (int)OFF[r - 1]) : 0; };
    store_all((dir == 0 ? tmp.orp : tmp.irp) + nslot, G + 1, row_start);
    if (nd == 2) store_all(tmp.irp + nslot, G + 1, [&](int g) { return row_start(G + g) - Ec; });
    block_sync<kLds>();
  }
  if (t == 0) {
    tmp.Gc[c] = G;
    tmp.Ec[c] = Ec;
  }
}

extern __shared__ __attribute__((aligned(16))) char dc_smem[];

// The candidates whose working set is larger than `above` and at most `most`; `lds` bytes are there.  kBatch: places that a
// thread takes together, so that their latencies overlap.
template <int kBatch>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 8))) void contract_kernel(
    BaseGraphs bg, int C, const int* cand_graph, const int* cand_off, const int* label, ContractTmp tmp, int* new_id_out,
    int* status, int above, int most, int lds) {
  __shared__ int wsum[20];
  if (call_failed(status)) return;
  for (int c = blockIdx.x; c < C; c += gridDim.x) {
    const int b = cand_graph[c], coff = cand_off[c], eslot = tmp.tmp_eoff[c];
    const int N = bg.gno[b + 1] - bg.gno[b];
    const int E = bg.geo[b + 1] - bg.geo[b];
    const int need = slab_need(N, E);
    if (need <= above || need > most) continue;
    const Slab L = slab_layout(N, E, lds);
    contract_one<true, u16, kBatch>(bg, c, b, N, E, dc_smem, L, Places{}, 0, coff, eslot, label, tmp, new_id_out, status, wsum);
    __syncthreads();
  }
}

// Where a base graph does not fit LDS, its candidates and those that need a CU's LDS to themselves (all of them where there
// are few): they are few and long and differ several times in size, and are handed out one at a time, largest
// first (the order prep_kernel leaves), through a counter.  55 candidates of 55 graphs of 2 to 21 k nodes, four of which do not fit: 417 us in
// launches of their own after the others, 244 us.
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 8))) void contract_large_kernel(
    BaseGraphs bg, const int* cand_graph, const int* cand_off, const int* label, ContractTmp tmp, int* new_id_out, int* status,
    char* gslab, size_t slab_stride, int most, int lds) {
  __shared__ int wsum[20];
  __shared__ int next_item;
  if (call_failed(status)) return;
  const int n_big = tmp.big_meta[0];
  for (;;) {
    if (threadIdx.x == 0) next_item = atomicAdd(&tmp.big_meta[1], 1);
    __syncthreads();
    const int i = next_item;
    __syncthreads();                          // everyone has read it before thread 0 writes the next one
    if (i >= n_big) break;
    const int c = tmp.big_order[i];
    const int b = cand_graph[c], coff = cand_off[c], eslot = tmp.tmp_eoff[c];
    const int N = bg.gno[b + 1] - bg.gno[b];
    const int E = bg.geo[b + 1] - bg.geo[b];
    const Places places{dc_smem, dc_smem + lds, gslab + (size_t)blockIdx.x * slab_stride};
    if (slab_need(N, E) <= most)
      contract_one<true, u16, 8>(bg, c, b, N, E, dc_smem, slab_layout(N, E, lds), Places{}, 0, coff, eslot, label, tmp, new_id_out, status, wsum);
    else if (E <= 65535) contract_one<false, u16, 8>(bg, c, b, N, E, nullptr, Slab{}, places, lds, coff, eslot, label, tmp, new_id_out, status, wsum);
    else contract_one<false, int, 8>(bg, c, b, N, E, nullptr, Slab{}, places, lds, coff, eslot, label, tmp, new_id_out, status, wsum);
    __syncthreads();
  }
}

// Clears the call's status, validates the candidate list and scans the base edge counts (one workgroup).
__global__ __launch_bounds__(1024) void prep_kernel(BaseGraphs bg, int C, const int* cand_graph, const int* cand_off,
                                                     int* tmp_eoff, long long max_base_nodes,
                                                     long long max_base_edges, int* status, int* big_order,
                                                     int* big_meta, int order_above, int max_weight) {
  __shared__ int wsum[16];
  const int t = threadIdx.x, T = blockDim.x;
  int bad = 0;
  if (t == 0) status[0] = 0;                  // a call begins here (a launch of its own for this was 4 us)
  for (int c = t; c < C; c += T) {
    const int b = cand_graph[c];
    int e = 0;
    if (b < 0 || b >= bg.n_graphs) {
      bad = 1;
    } else {
      const int n = bg.gno[b + 1] - bg.gno[b];
      if (cand_off[c + 1] - cand_off[c] != n) bad = 1;
      e = bg.geo[b + 1] - bg.geo[b];
    }
    tmp_eoff[c] = e;
  }
  if (t == 0 && cand_off[0] != 0) bad = 1;
  bad = __syncthreads_or(bad);
  if (bad) {
    if (t == 0) set_error(status, (int)DC_ERR_BAD_PARTITION);
    return;
  }
  // 64-bit check of the edge total before the 32-bit scan
  long long es = 0;
  for (int c = t; c < C; c += T) es += tmp_eoff[c];
  __shared__ long long esum[16];
  for (int o = 32; o > 0; o >>= 1) es += __shfl_down(es, o, 64);
  if ((t & 63) == 0) esum[t >> 6] = es;
  __syncthreads();
  long long tot = 0;
  for (int i = 0; i < (T >> 6); ++i) tot += esum[i];
  if (tot > max_base_edges || (long long)cand_off[C] > max_base_nodes) {
    if (t == 0) set_error(status, (int)DC_ERR_CAPACITY);
    return;
  }
  const int total = block_exscan(tmp_eoff, tmp_eoff, C, wsum);
  if (t == 0) tmp_eoff[C] = total;
  if (order_above == INT_MAX) return;         // every base graph fits LDS
  // The candidates whose base graph needs more LDS than `order_above`, in sixteen classes of size (nodes and edges), largest
  // class first (the order inside a class is whatever the atomics give: it decides which workgroup contracts a
  // candidate, not what is written).
  __shared__ int hist[16], base[16];
  if (t < 16) hist[t] = 0;
  __syncthreads();
  auto size_class = [&](int c) {
    const int b = cand_graph[c], N = bg.gno[b + 1] - bg.gno[b], E = bg.geo[b + 1] - bg.geo[b];
    return slab_need(N, E) <= order_above ? -1 : (int)(((long long)N + E) * 15 / max_weight);
  };
  for (int c = t; c < C; c += T) {
    const int k = size_class(c);
    if (k >= 0) atomicAdd(&hist[k], 1);
  }
  __syncthreads();
  if (t == 0) {
    int run = 0;
    for (int k = 15; k >= 0; --k) {
      base[k] = run;
      run += hist[k];
    }
    big_meta[0] = run;
    big_meta[1] = 0;
  }
  __syncthreads();
  for (int c = t; c < C; c += T) {
    const int k = size_class(c);
    if (k >= 0) big_order[atomicAdd(&base[k], 1)] = c;
  }
}

// Scans contracted sizes over the batch and checks the output capacities.
__global__ __launch_bounds__(1024) void scan_sizes_kernel(int C, const int* Gc, const int* Ec, int* node_off,
                                                           int* edge_off, long long cap_nodes, long long cap_edges,
                                                           int* status, int* totals) {
  __shared__ int wsum[16];
  if (status[0] != 0) return;
  const int nt = block_exscan(Gc, node_off, C, wsum);
  const int et = block_exscan(Ec, edge_off, C, wsum);
  if (threadIdx.x == 0) {
    node_off[C] = nt;
    edge_off[C] = et;
    totals[0] = nt;
    totals[1] = et;
    if (nt > cap_nodes || et > cap_edges) set_error(status, (int)DC_ERR_CAPACITY);
  }
}


// Up to this many candidates finalize_kernel sums the sizes in front of its candidate itself (one per thread) instead of
// after a scan kernel: one launch of 4 us less in passes of 50 to 350 us.
constexpr int kOwnScan = 256;

// dst[i] = add + src[i], i < n, by T threads: four entries a load and a store
__device__ __forceinline__ void copy_add(int* dst, const int* src, int n, int add, int t, int T) {
  struct __attribute__((packed, aligned(4))) Quad { int x[4]; };
  const int n4 = n >> 2;
  for (int i = t; i < n4; i += T) {
    const Quad q = *reinterpret_cast<const Quad*>(src + 4 * i);
    store4(dst + 4 * i, add + q.x[0], add + q.x[1], add + q.x[2], add + q.x[3]);
  }
  for (int i = 4 * n4 + t; i < n; i += T) dst[i] = add + src[i];
}

// Places candidate c's lists at their block-diagonal position and sums features.  gridDim.y workgroups share a
// candidate: they take its list entries and feature items in turn.
template <bool kBf16>
__global__ __launch_bounds__(256) void finalize_kernel(BaseGraphs bg, int C, const int* cand_graph,
                                                        const int* cand_off, ContractTmp tmp, BatchView out, int F,
                                                        int* status, int* totals) {
  if (C > kOwnScan && status[0] != 0) return;        // set by an earlier launch only
  const int c = blockIdx.x, t = blockIdx.y * blockDim.x + threadIdx.x, T = gridDim.y * blockDim.x;
  const int b = cand_graph[c];
  const int coff = cand_off[c];
  const int nslot = coff + c, eslot = tmp.tmp_eoff[c];
  const int G = tmp.Gc[c], E = tmp.Ec[c];
  int n0, e0;
  if (C <= kOwnScan) {
    __shared__ int wn[4], we[4], own[2], failed;
    if (threadIdx.x == 0) failed = status[0];        // read once: workgroup 0 of this launch may set it
    const int i = threadIdx.x, lane = i & 63, wave = i >> 6;
    const int xn = i < C ? tmp.Gc[i] : 0, xe = i < C ? tmp.Ec[i] : 0;
    int sn = wave_incl_scan(xn), se = wave_incl_scan(xe);
    if (lane == 63) {
      wn[wave] = sn;
      we[wave] = se;
    }
    __syncthreads();
    if (failed) return;
    int nt = 0, et = 0;
    for (int w = 0; w < 4; ++w) {
      if (w < wave) {
        sn += wn[w];
        se += we[w];
      }
      nt += wn[w];
      et += we[w];
    }
    if (i == c) {
      own[0] = sn - xn;
      own[1] = se - xe;
    }
    const bool fits = nt <= out.cap_nodes && et <= out.cap_edges;
    if (blockIdx.x == 0 && blockIdx.y == 0) {
      if (i < C) {
        out.node_off[i] = sn - xn;
        out.edge_off[i] = se - xe;
      }
      if (i == 0) {
        out.node_off[C] = nt;
        out.edge_off[C] = et;
        totals[0] = nt;
        totals[1] = et;
        if (!fits) set_error(status, (int)DC_ERR_CAPACITY);
      }
    }
    __syncthreads();
    if (!fits) return;
    n0 = own[0];
    e0 = own[1];
  } else {
    n0 = out.node_off[c];
    e0 = out.edge_off[c];
  }
  const int gend = (c == C - 1) ? G + 1 : G;   // the last candidate also writes the closing entry
  copy_add(out.out_rowptr + n0, tmp.orp + nslot, gend, e0, t, T);
  copy_add(out.in_rowptr + n0, tmp.irp + nslot, gend, e0, t, T);
  copy_add(out.out_col + e0, tmp.oc + eslot, E, n0, t, T);
  copy_add(out.in_col + e0, tmp.ic + eslot, E, n0, t, T);
  // feature sums: members in ascending base index, fp32 accumulation, one rounding.  A thread works on
  // four (group, column quad) items at a time, so that the dependent loads of an item (list bounds,
  // member numbers, member rows) overlap with those of three others: the loop is bound by memory latency.
  const int q = F >> 2;
  const float4* X4 = reinterpret_cast<const float4*>(bg.X) + (size_t)bg.gno[b] * q;
  const int* ms = tmp.mstart + nslot;
  const int* mem = tmp.members + coff;
  const int items = G * q;
  for (int i0 = t; i0 < items; i0 += 4 * T) {
    int f[4], m[4], me[4], g[4];
    float4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = i0 + j * T;
      const bool ok = i < items;
      g[j] = ok ? i / q : 0;
      f[j] = ok ? i - g[j] * q : 0;
      m[j] = ok ? ms[g[j]] : 0;
      me[j] = ok ? ms[g[j] + 1] : 0;
      acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // rounds of up to two members per item, the four items' loads in flight together; the member numbers of the
    // next round are asked for together with the rows of this one, so that a round costs one memory round trip
    int i0m[4], i1m[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      i0m[j] = m[j] < me[j] ? mem[m[j]] : -1;
      i1m[j] = m[j] + 1 < me[j] ? mem[m[j] + 1] : -1;
    }
    bool more = true;
    while (more) {
      float4 x0[4], x1[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        x0[j] = i0m[j] >= 0 ? X4[(size_t)i0m[j] * q + f[j]] : make_float4(0.f, 0.f, 0.f, 0.f);
        x1[j] = i1m[j] >= 0 ? X4[(size_t)i1m[j] * q + f[j]] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
      int n0m[4], n1m[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        n0m[j] = m[j] + 2 < me[j] ? mem[m[j] + 2] : -1;
        n1m[j] = m[j] + 3 < me[j] ? mem[m[j] + 3] : -1;
      }
      more = false;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        // added in member order; a member that does not exist adds nothing (not even +0 to a -0 sum)
        if (i0m[j] >= 0) { acc[j].x += x0[j].x; acc[j].y += x0[j].y; acc[j].z += x0[j].z; acc[j].w += x0[j].w; }
        if (i1m[j] >= 0) { acc[j].x += x1[j].x; acc[j].y += x1[j].y; acc[j].z += x1[j].z; acc[j].w += x1[j].w; }
        m[j] += 2;
        more |= m[j] < me[j];
        i0m[j] = n0m[j];
        i1m[j] = n1m[j];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = i0 + j * T;
      if (i >= items) continue;
      const size_t row = (size_t)(n0 + g[j]);
      if (kBf16) {
        uint2 p;
        p.x = pack_bf16x2(acc[j].x, acc[j].y);
        p.y = pack_bf16x2(acc[j].z, acc[j].w);
        reinterpret_cast<uint2*>(out.Xc)[row * q + f[j]] = p;
      } else {
        reinterpret_cast<float4*>(out.Xc)[row * q + f[j]] = acc[j];
      }
    }
  }
}

}  // namespace

int contract_size_class(int n_nodes, int n_edges, int lds_limit) {
  const int need = slab_need(n_nodes, n_edges);
  for (int k = 0; k < kSizeClasses; ++k)
    if (need <= size_class_of(k, lds_limit).most) return k;
  return kSizeClasses;
}
size_t contract_slab_bytes(int n_nodes, int n_edges) { return slab_bytes(n_nodes, n_edges); }

__global__ void reset_status_kernel(int* status) { status[0] = 0; }

hipError_t launch_contract(const ContractLaunch& a, Profiler* prof, hipStream_t s) {
  if (a.n_cand <= 0) {
    hipLaunchKernelGGL(reset_status_kernel, dim3(1), dim3(1), 0, s, a.status);
    return hipGetLastError();
  }
  const int C = a.n_cand;
  // Classes of few candidates need not follow each other: with a CU for every candidate, or every two where there are several
  // classes, one launch takes all (25 candidates of 25 graphs of 0.2 to 3.2 k nodes: 73 us in two launches, 45 us; 280 of 40
  // of 0.3 to 6 k 162 and 82 us; 512 of 64 of 0.5 to 3.5 k 122 and 107 us).
  const bool beyond = (a.size_classes >> kSizeClasses) & 1, several = a.size_classes & (a.size_classes - 1);
  const bool alone = C <= (several ? 2 : 1) * a.n_cu;
  const int order_above = !beyond ? INT_MAX : alone ? 0 : size_class_of(kSizeClasses - 2, a.lds_limit).most;
  if (prof) prof->begin(kFamPrep, s);
  hipLaunchKernelGGL(prep_kernel, dim3(1), dim3(1024), 0, s, a.bg, C, a.cand_graph, a.cand_off, a.tmp.tmp_eoff,
                     a.max_base_nodes, a.max_base_edges, a.status, a.tmp.big_order, a.tmp.big_meta, order_above,
                     (int)std::min<long long>((long long)a.max_graph_nodes + a.max_graph_edges, INT_MAX));
  if (prof) prof->end(s);
  if (prof) prof->begin(kFamContract, s);
  if (beyond)
    hipLaunchKernelGGL(contract_large_kernel, dim3(C < a.slab_wgs ? C : a.slab_wgs), dim3(1024), a.lds_limit, s, a.bg, a.cand_graph,
                       a.cand_off, a.group_id, a.tmp, a.out.new_id, a.status, a.slab, a.slab_stride,
                       size_class_of(kSizeClasses - 1, a.lds_limit).most, a.lds_limit);
  int above = 0;
  for (int k = 0; k < kSizeClasses; ++k) {
    const SizeClass z = size_class_of(k, a.lds_limit);
    if (alone ? !beyond && (a.size_classes >> k) == 1 : ((a.size_classes >> k) & 1) && !(beyond && k == kSizeClasses - 1)) {
      // a workgroup that has its CU to itself takes as many waves as there are nodes for
      const int threads = C <= a.n_cu && a.max_graph_nodes > 512 ? 1024 : z.threads;
      const bool small = a.max_graph_nodes <= threads;
      hipLaunchKernelGGL((small ? contract_kernel<2> : contract_kernel<8>), dim3(C), dim3(threads), z.lds, s, a.bg, C,
                         a.cand_graph, a.cand_off, a.group_id, a.tmp, a.out.new_id, a.status, above, z.most, z.lds);
    }
    if (!alone) above = z.most;
  }
  if (prof) prof->end(s);
  if (prof) prof->begin(kFamFinalize, s);
  if (C > kOwnScan) hipLaunchKernelGGL(scan_sizes_kernel, dim3(1), dim3(1024), 0, s, C, a.tmp.Gc, a.tmp.Ec, a.out.node_off,
                     a.out.edge_off, a.out.cap_nodes, a.out.cap_edges, a.status, a.totals);
  // One workgroup per candidate fills the chip once there are eight of them per CU.  With fewer candidates several
  // share one, down to one round of 4 x 256 feature items each (7 candidates of 1.4 k groups and F = 64: 111 us with
  // one workgroup each, 9.8 us with 23).
  const int rounds = ceil_div(a.max_graph_nodes * (a.F > 4 ? a.F >> 2 : 1), 4 * 256);
  const int want = ceil_div(8 * a.n_cu, C);
  const dim3 fgrid(C, want < rounds ? want : (rounds > 0 ? rounds : 1));
  if (a.bf16)
    hipLaunchKernelGGL(finalize_kernel<true>, fgrid, dim3(256), 0, s, a.bg, C, a.cand_graph, a.cand_off, a.tmp,
                       a.out, a.F, a.status, a.totals);
  else
    hipLaunchKernelGGL(finalize_kernel<false>, fgrid, dim3(256), 0, s, a.bg, C, a.cand_graph, a.cand_off, a.tmp,
                       a.out, a.F, a.status, a.totals);
  if (prof) prof->end(s);
  return hipGetLastError();
}

hipError_t contract_set_lds_limit(int bytes) {
  for (const void* k : {reinterpret_cast<const void*>(&contract_kernel<8>), reinterpret_cast<const void*>(&contract_kernel<2>),
                        reinterpret_cast<const void*>(&contract_large_kernel)}) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace dc
