// End-to-end time of a candidate module by list scheduling (Sec. 3.4; gfx950).
//
// Computation ops run one at a time on one device in the order of a FIFO ready queue (an
// op enters the tail when its last dependency clears; it starts when the device is free
// and its predecessors are done).  All-reduce instructions run one at a time on a
// communication channel, in the order in which their tensors are produced, each starting
// when its tensor is produced and the channel is clear, for T = C x + D (Sec. 3.1,
// Profiler); they overlap with computation.  The result is the later of the two ends.
// Where the text is silent: the queue starts with the source ops in ascending index; an
// all-reduce goes on the channel the moment its last predecessor is processed, before the
// next op is taken, ties in ascending index; successors are released in ascending index;
// a module whose graph has a cycle (an invalid fusion) costs +infinity.
//
// Times are fp64, added in the order the rules fix, so the result does not depend on the
// implementation.
//
//   simulate_order_kernel    modules whose execution times are not negative and whose all-reduces
//                            have no successors: the order of the nodes does not depend on the times
//                            there and is found by all nodes at once; the times are added along it
//   simulate_walk_kernel     the others, where an op waits for an all-reduce (a weight update behind
//                            its tensor) or a time is negative: one wave walks the module node by
//                            node, with its arrays in LDS; the lanes release the successors of the
//                            current node together (lists are duplicate free, so no two lanes touch
//                            one node) and append the newly ready ones in lane order = ascending
//                            index
//   simulate_walk_global_kernel  those too large for LDS, in slices of global memory
#include <math.h>

#include <mutex>

#include "common.h"

namespace dc {
namespace {

// The arrays of a module that is walked, in global memory ...
__host__ __device__ inline size_t sim_bytes(long long G, long long E) {
  // ready[G] f64 | val[G] f32 | dep[G] i32 | queue[G] i32 | rp[G+1] i32 | ci[E] u16 (padded to 8 bytes)
  return (size_t)G * (8 + 4 + 4 + 4) + (size_t)(G + 1) * 4 + (((size_t)E * 2 + 7) & ~(size_t)7) + 8;
}
// ... and in LDS, where a byte saved is a module more per CU: dependency counters and queue entries of 16 bits
// (a module has fewer than 65536 nodes; the counter keeps bit 15 for the all-reduce flag, so it takes modules
// of up to 32768 nodes, more than LDS holds anyway).
__host__ __device__ inline size_t sim_lds_bytes(long long G, long long E) {
  // ready[G] f64 | val[G] f32 | rp[G+1] i32 | dep[G] u16 | queue[G] u16 | ci[E] u16 (padded to 8 bytes)
  if (G > 32768) return ~(size_t)0;
  return (size_t)G * (8 + 4) + (size_t)(G + 1) * 4 + (((size_t)G * 4 + (size_t)E * 2 + 7) & ~(size_t)7) + 8;
}
template <bool kLds>
struct SimTypes {                 // global memory
  typedef int dep_t;
  typedef int q_t;
  static constexpr int kAr = 1 << 30;      // flag in the dependency counter: the node is an all-reduce
};
template <>
struct SimTypes<true> {           // LDS
  typedef unsigned short dep_t;
  typedef unsigned short q_t;
  static constexpr int kAr = 1 << 15;
};

// Modules that the first kernel leaves to the walk carry this pattern in their cost: a NaN that no arithmetic gives.
constexpr unsigned kLeft = 0x7FC5A11Du;

extern __shared__ __attribute__((aligned(16))) char dc_sim_smem[];

// ---------------------------------------------------------------------------------------------------
// The order of a module by iteration, its times along the order.
//
// With execution times that are not negative the device's clock never runs backwards, so an op never waits for its
// predecessors (they ran before it) and starts when the device is free; an all-reduce without successors holds
// nothing up.  The order of the ops is then a matter of the graph alone: an op enters the queue when its last
// predecessor ends, so the ops stand in the order of (place of the last predecessor, index), where the place of an op
// is its rank in that same order.  The kernel solves this by iteration: from any places it computes every op's key =
// the largest place among its predecessors, sorts by (key, index) and takes the ranks as the new places, until
// nothing changes.  A fixed point in which every key lies before its op's place is the order of the queue: by
// induction over the places, the first k ops are the queue's, and the next one is the smallest (key, index) among the
// ops whose predecessors are all among them.  For the same reason the places before the first one that changed or
// holds a key not before it are right from then on and grow by one a round at the least; where no op outside them has
// all its predecessors among them, the module has a cycle.
//
// One iteration is parallel over all nodes, where the walk that this replaces took the nodes one after another at
// four dependent LDS round trips each (about 800 cycles a node).  The number of iterations is the depth to which
// neighbouring chains interleave, not the length of the module: from the index order as the first guess 4 to 7 on the
// contracted modules of a 24-block transformer (1.4 k nodes, 1.3 k of them one after another), 13 on the unfused
// module (6.6 k nodes), 20 to 36 on power-law graphs.
//
// Where chains that run side by side are numbered one after the other (two towers, long branches), or the numbering
// follows no order, that depth is the length of the chains.  So after sixteen rounds, unless at their rate as many more
// are enough, the depth of every op is found and ranks by (depth, index) are the second guess: an op of smaller depth
// always comes first.  Depths by iteration too: every op chooses a predecessor, pointer doubling gives the lengths of the
// paths along the chosen ones, and ops with a deeper predecessor choose that; two to four steps of a few rounds each.  A
// path longer than the module has nodes is a cycle.
// Mostly one round then settles the rest (two chains of 300 ops, 4096 modules: 4.4 ms by rounds, 0.33 now, 0.63 by the
// walk; two unfused modules of 1.6 k nodes side by side, 1000 times: 6.4, 0.53, 2.5).  What is still slow is left to the
// walk: branches numbered at random, whose order settles depth by depth (16 and 8 rounds in vain: a quarter of the walk).
//
// A thread owns NPT nodes and keeps their predecessors (three or four each; what longer lists hold beyond three lies
// in LDS, or is read from memory again once that is full) and keys in registers; LDS holds the places, the counters of
// the sort and the order: 8 bytes per node with the longer lists.  The sort is a counting sort by key (16-bit counters,
// two to a word); equal keys are the ops that one op releases, and an op finds its rank among them by comparing with
// each.  Where one op has more than kTies successors (or tensors without predecessors are about), that could take the
// square of their number: there the nodes of such a key are marked in a bitmap, one key after another, and the bits
// below a node give its rank.  One op that releases 6 k others, 512 modules: 6.6 ms by comparing, 3.1 now, 5.8 by the
// walk; 6 k tensors of one op: 5.1, 1.3, 2.7.  Whether a module is so wide is seen when it is loaded: looked for in
// every round it would cost the others 3 %.  Sources keep their places throughout.
//
// The times: the device's clock is a running sum over the ops, the channel's a chain of maximum and sum over the
// all-reduces, which are sorted by (place of the last predecessor, index) in the same way and taken by one wave.
//
// What bounds it: LDS round trips between some six barriers a round (about 15 k cycles a round with 1024 threads and
// 6.6 k nodes, 12 rounds, and 60 k for the times; 64 or 256 threads for small modules: 9 k a round).  Measured, walk
// before -> now: 4096 contracted modules of 1.4 k nodes 2.48 -> 0.24 ms, 1000 nearly unfused ones of 6.5 k nodes
// (walked in global memory before) 6.02 -> 0.47 ms, 16 modules of 0.7 k nodes 0.27 -> 0.03 ms.  Workgroups of 512
// threads with sixteen nodes each, two per CU, take the same time as 1024 with eight.
// ---------------------------------------------------------------------------------------------------
constexpr int kSecondGuess = 16;       // so many more rounds take longer than a second guess
constexpr int kGuessRound = 1 << 16;   // the number of the round that takes it
constexpr int kMostSteps = 4;          // of the second guess
constexpr int kWalkRounds = 64;        // the walk takes as long as so many rounds, and one more for 32 nodes
constexpr int kTies = 128;             // up to so many, comparing is cheaper than four barriers for a key
constexpr int kNone = 0x7FFFFFFF;

__device__ __forceinline__ int lane_of(int x, int l) { return __builtin_amdgcn_readlane(x, l); }
__device__ __forceinline__ double lane_of(double x, int l) {
  const long long b = __double_as_longlong(x);
  const unsigned lo = (unsigned)lane_of((int)b, l), hi = (unsigned)lane_of((int)(b >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <int T, int NPT>
struct OrderLds {
  static constexpr int kCap = T * NPT;
  static constexpr int kPlace = 0;                                   // u16 [kCap + 1]: place + 1; entry kCap is 0
  static constexpr int kOrder = (2 * (kCap + 1) + 15) & ~15;         // u16 [kCap]
  static constexpr int kCount = kOrder + ((2 * kCap + 15) & ~15);    // u16 [kCap + 2]: counters by key, then starts
  static constexpr int kExtra = kCount + ((2 * (kCap + 2) + 15) & ~15);   // u16 [kCap]: predecessors of longer lists
  static constexpr int kSums = kExtra + ((2 * kCap + 15) & ~15);     // f64 [max(T, 128)]: see the times
  static constexpr int kValue = kCount;                              // f32 [kCap]: times along the order, at last
  static_assert(kSums - kValue >= 4 * kCap, "the times take the place of the counters and the longer lists");
  static constexpr int kBytes = kSums + 8 * (T > 128 ? T : 128);
  static constexpr int kPath = kOrder;                               // u32 [kCap], between two rounds: see depths
  static_assert(kExtra - kPath >= 4 * kCap, "the paths take the place of the order and the counters");
  static constexpr int kWords = kCap / 32;                           // bitmap of the nodes, while no sums are kept
  static_assert(kWords * 6 <= 8 * (T > 128 ? T : 128), "u32 [kWords] bits, u16 [kWords] bits set before each word");
};

// Exclusive scan of the counters of keys 1 .. n (16 bits each, at words [0, words)) in place, starting from `base`;
// counter 0 becomes `base`.  Ends with a barrier.
template <int T>
__device__ __forceinline__ void scan_counts(unsigned* words_, int words, int base, int* wsum) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int K = (words + T - 1) / T;
  const int lo = min(t * K, words), hi = min(lo + K, words);
  int s = 0;
  for (int i = lo; i < hi; ++i) s += (int)(words_[i] & 0xFFFFu) + (int)(words_[i] >> 16);
  const int inc = wave_incl_scan(s);
  int run = base + inc - s;
  if constexpr (T > 64) {
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < T / 64; ++w) {
      const int x = wsum[w];
      run += w < wave ? x : 0;
    }
  }
  for (int i = lo; i < hi; ++i) {
    const unsigned x = words_[i];
    const int mid = run + (int)(x & 0xFFFFu);
    words_[i] = (unsigned)run | (unsigned)mid << 16;
    run = mid + (int)(x >> 16);
  }
  __syncthreads();
}

template <int T, int NPT>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(T == 64 ? 5 : 4, 8))) void simulate_order_kernel(
    const int* __restrict__ node_off, const int* __restrict__ out_rp, const int* __restrict__ in_rp,
    const int* __restrict__ in_ci, const float* __restrict__ op_time, const float* __restrict__ ar_size, int C,
    float ar_c, float ar_d, float* __restrict__ cost, int fewest, int last, const int* __restrict__ status) {
  // the modules of `fewest` to T * NPT nodes; the last class to be launched leaves the larger ones to the walk
  typedef OrderLds<T, NPT> Lds;
  constexpr int kCap = Lds::kCap, kWaves = T / 64;
  __shared__ int wsum[kWaves], sh_min[2][2], sh_src[NPT][kWaves], n_extra, n_tied, sh_wide;
  __shared__ unsigned short tied[kCap / kTies];
  unsigned short* place = reinterpret_cast<unsigned short*>(dc_sim_smem + Lds::kPlace);
  unsigned* count2 = reinterpret_cast<unsigned*>(dc_sim_smem + Lds::kCount);
  unsigned short* count = reinterpret_cast<unsigned short*>(dc_sim_smem + Lds::kCount);
  unsigned short* order = reinterpret_cast<unsigned short*>(dc_sim_smem + Lds::kOrder);
  unsigned short* extra = reinterpret_cast<unsigned short*>(dc_sim_smem + Lds::kExtra);
  float* value = reinterpret_cast<float*>(dc_sim_smem + Lds::kValue);
  double* sums = reinterpret_cast<double*>(dc_sim_smem + Lds::kSums);
  if (status[0] != 0) return;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  for (int c = blockIdx.x; c < C; c += gridDim.x) {
    const int n0 = node_off[c], G = node_off[c + 1] - n0;
    if (G < fewest) continue;
    if (G > kCap) {
      if (last && t == 0) cost[c] = __uint_as_float(kLeft);
      continue;
    }
    if (t == 0) n_extra = sh_wide = 0;
    __syncthreads();
    // ---- the thread's nodes t, t + T, ...: predecessors, kind
    unsigned p01[NPT], p23[NPT];
    unsigned is_op = 0, is_ar = 0, is_src = 0, more = 0, far = 0;   // bit i: node t + i * T
    bool plain = true, wide = false;                         // wide: more than kTies nodes may share a key
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const int v = t + i * T;
      p01[i] = p23[i] = 2u * kCap * 0x10001u;                // twice the numbers: where their places lie
      if (v < G) {
        // (all six requested together, whatever the node: one wait)
        const int a = in_rp[n0 + v], d = in_rp[n0 + v + 1] - a;
        const int released = out_rp[n0 + v + 1] - out_rp[n0 + v];
        const float size = ar_size[n0 + v], time = op_time[n0 + v];
        const bool ar = size >= 0.0f;
        plain &= (ar & (released == 0)) | (!ar & (time >= 0.0f));   // a NaN is neither
        wide |= released > kTies || (ar && d == 0);
        const unsigned x0 = d > 0 ? in_ci[a] - n0 : kCap, x1 = d > 1 ? in_ci[a + 1] - n0 : kCap;
        const unsigned x2 = d > 2 ? in_ci[a + 2] - n0 : kCap;
        unsigned x3 = d > 3 ? in_ci[a + 3] - n0 : kCap;
        if (d > 4) {                                           // the others follow each other in LDS, kCap ends them
          const int at = atomicAdd(&n_extra, d - 2);
          if (at + d - 2 <= kCap) {
            extra[at] = (unsigned short)x3;
            for (int k = 4; k < d; ++k) extra[at + k - 3] = (unsigned short)(in_ci[a + k] - n0);
            extra[at + d - 3] = (unsigned short)kCap;
            x3 = (unsigned)at;
            more |= 1u << i;
          } else {
            far |= 1u << i;
          }
        }
        p01[i] = 2 * x0 | x1 << 17;
        p23[i] = 2 * x2 | x3 << ((more >> i) & 1u ? 16 : 17);
        is_ar |= (unsigned)ar << i;
        is_op |= (unsigned)!ar << i;
        is_src |= (unsigned)(!ar && d == 0) << i;
        place[v] = (unsigned short)(v + 1);                  // the first guess: the index order
      }
    }
    if (t == 0) place[kCap] = 0;
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const unsigned long long m = __ballot((is_src >> i) & 1u);
      if (lane == 0) sh_src[i][wave] = __popcll(m);
    }
    if (t == 0) sh_min[0][0] = sh_min[0][1] = kNone;
    if (__any(wide) && lane == 0) sh_wide = 1;
    if (__syncthreads_or(!plain)) {
      if (t == 0) cost[c] = __uint_as_float(kLeft);
      continue;
    }
    const bool ties = __builtin_amdgcn_readfirstlane(sh_wide) != 0;
    // sources stand first, in index order
    int n_src = 0;
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const unsigned long long m = __ballot((is_src >> i) & 1u);
      int before = n_src;
      for (int w = 0; w < kWaves; ++w) {
        const int k = sh_src[i][w];
        if (w < wave) before += k;
        n_src += k;
      }
      if ((is_src >> i) & 1u) place[t + i * T] = (unsigned short)(before + __popcll(m & ((1ull << lane) - 1ull)) + 1);
    }
    const int words = (G + 3) >> 1;                          // counters of keys 0 .. G and one more start

    // f(twice the predecessor) for those of node i, of kCap where there are fewer than four
    auto each_before = [&](int i, auto&& f) {
      // (kept from being taken out of the loop of rounds: unpacked, the predecessors would take four registers a node, and
      // the bits of all nodes more scalar registers than there are)
      asm volatile("" : "+v"(p01[i]), "+v"(p23[i]), "+v"(more), "+v"(far));
      f(p01[i] & 0xFFFFu);
      f(p01[i] >> 16);
      f(p23[i] & 0xFFFFu);
      if ((more >> i) & 1u) {
        for (int at = p23[i] >> 16, u = extra[at]; u != kCap; u = extra[++at]) f(2u * u);
      } else {
        f(p23[i] >> 16);
      }
      if ((far >> i) & 1u) {
        int v = n0 + t + i * T;
        asm volatile("" : "+v"(v));
        for (int e = in_rp[v] + 4; e < in_rp[v + 1]; ++e) f(2u * (in_ci[e] - n0));
      }
    };
    auto place_at = [&](unsigned twice) { return *reinterpret_cast<const unsigned short*>(dc_sim_smem + Lds::kPlace + twice); };
    // key of node i: the largest place + 1 among its predecessors
    auto key_of = [&](int i) {
      int k = 0;
      each_before(i, [&](unsigned twice) { k = max(k, (int)place_at(twice)); });
      return k;
    };
    // Sorts the nodes of the mask by (key, index), ranks counted from `base`; order[off + base] and the places behind
    // it serve as scratch.  ka[i]: key of the thread's node i, and above it its turn among those of the same key.
    unsigned ka[NPT];
    auto sort = [&](unsigned mask, int base, int off) {
      for (int i = t; i < words; i += T) count2[i] = 0;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NPT; ++i)
        if ((mask >> i) & 1u) {
          const int key = key_of(i), sh = (key & 1) << 4;
          ka[i] = (unsigned)key | ((atomicAdd(&count2[key >> 1], 1u << sh) >> sh) << 16);
        }
      __syncthreads();
      scan_counts<T>(count2, words, base, wsum);
#pragma unroll
      for (int i = 0; i < NPT; ++i)
        if ((mask >> i) & 1u) order[off + count[ka[i] & 0xFFFFu] + (ka[i] >> 16)] = (unsigned short)(t + i * T);
      __syncthreads();
    };
    auto rank_of = [&](int i, int off) {
      const int s = count[ka[i] & 0xFFFFu], e = count[(ka[i] & 0xFFFFu) + 1];
      int r = s;
      if (e - s > 1)
        for (int k = s; k < e; ++k) r += (int)order[off + k] < t + i * T;
      return r;
    };
    // the same for a wide module: f(node, rank, key) for all sorted nodes.  Here a thread takes places of the scratch
    // order, not its own nodes (which would cost the usual module registers), and looks for the key of each.
    auto tied_ranks = [&](int base, int off, auto&& f) {
      if (t == 0) n_tied = 0;
      __syncthreads();
      for (int k = base + t; k < (int)count[G + 1]; k += T) {
        int key = 0;                                         // the last key that starts at or before k
        for (int hi = G + 1; hi - key > 1;) {
          const int mid = (key + hi) >> 1;
          if ((int)count[mid] <= k) key = mid;
          else hi = mid;
        }
        const int s = count[key], e = count[key + 1], v = order[off + k];
        if (e - s <= kTies) {
          int r = s;
          for (int j = s; j < e; ++j) r += (int)order[off + j] < v;
          f(v, r, key);
        } else if (k == s) {
          tied[atomicAdd(&n_tied, 1)] = (unsigned short)key;
        }
      }
      __syncthreads();
      unsigned* bits = reinterpret_cast<unsigned*>(sums);
      unsigned short* below = reinterpret_cast<unsigned short*>(bits + Lds::kWords);
      const int n = n_tied;
#pragma unroll 1
      for (int q = 0; q < n; ++q) {
        const int key = tied[q], s = count[key], e = count[key + 1];
        for (int w = t; w < Lds::kWords; w += T) bits[w] = 0;
        __syncthreads();
        for (int k = s + t; k < e; k += T) atomicOr(&bits[order[off + k] >> 5], 1u << (order[off + k] & 31));
        __syncthreads();
        if (wave == 0) {
          constexpr int kPer = (Lds::kWords + 63) / 64;
          int c = 0;
          for (int w = lane * kPer; w < min((lane + 1) * kPer, Lds::kWords); ++w) c += __popc(bits[w]);
          int run = wave_incl_scan(c) - c;
          for (int w = lane * kPer; w < min((lane + 1) * kPer, Lds::kWords); ++w) {
            below[w] = (unsigned short)run;
            run += __popc(bits[w]);
          }
        }
        __syncthreads();
        for (int k = s + t; k < e; k += T) {
          const int v = order[off + k];
          f(v, s + below[v >> 5] + __popc(bits[v >> 5] & ((1u << (v & 31)) - 1u)), key);
        }
        __syncthreads();
      }
    };

    // The second guess: the depth of the ops in their places, so that the next round ranks them by (depth, index).
    // Returns whether it found a cycle.
    const unsigned mask = is_op & ~is_src;
    auto depths = [&]() {
      unsigned* path = reinterpret_cast<unsigned*>(dc_sim_smem + Lds::kPath);     // a node's ancestor, and its distance above
#pragma unroll 1
      for (int step = 0; step < kMostSteps; ++step) {
        // every op chooses its deepest predecessor (the first time the one that stands last)
        bool deeper = step == 0;
#pragma unroll
        for (int i = 0; i < NPT; ++i) {
          const int v = t + i * T;
          unsigned best = (unsigned)v;                       // place + 1 above the node
          if ((mask >> i) & 1u) {
            each_before(i, [&](unsigned twice) { best = max(best, (unsigned)place_at(twice) << 16 | twice >> 1); });
            deeper |= (best >> 16) >= (unsigned)place[v];
            best = (best & 0xFFFFu) | 0x10000u;
          }
          if (v < G) path[v] = best;
        }
        if (!__syncthreads_or(deeper)) return false;
        // the lengths of the paths along the chosen ones: a path reaches twice as far in every pass (the two halves of
        // a word belong together, so that it does not matter whether a pass finds another node's old or new word)
        bool on = true;
#pragma unroll 1
        for (int reach = 1; on; reach <<= 1) {
          if (reach >= 2 * G) return true;                   // so long a path from no source
          on = false;
#pragma unroll 4
          for (int i = 0; i < NPT; ++i) {
            const int v = min(t + i * T, G - 1);
            const unsigned x = path[v], y = path[x & 0xFFFFu];
            path[v] = min((x >> 16) + (y >> 16), (unsigned)(G - n_src)) << 16 | (y & 0xFFFFu);     // a cycle's grow on and on
            on |= y >> 16 != 0;
          }
          on = __syncthreads_or(on) != 0;
        }
#pragma unroll
        for (int i = 0; i < NPT; ++i)
          if ((mask >> i) & 1u) place[t + i * T] = (unsigned short)(n_src + (path[t + i * T] >> 16));
        __syncthreads();
      }
      return false;
    };

    // ---- the order of the ops
    int round = 0, state = 0;                                // 1: the order is found, 2: a cycle, 3: left to the walk
    int seen = 0;                                            // places that were right at the last look
    for (; state == 0; ++round) {
      sort(mask, n_src, 0);
      int changed = kNone, ahead = kNone;
      auto settle = [&](int v, int rank, int key) {
        if ((int)place[v] != rank + 1) {
          changed = min(changed, rank);
          place[v] = (unsigned short)(rank + 1);
        }
        if (key > rank) ahead = min(ahead, rank);
      };
      if (__builtin_expect(!ties && round != kGuessRound, 1)) {                   // depths may be shared by many in any module
#pragma unroll
        for (int i = 0; i < NPT; ++i)
          if ((mask >> i) & 1u) settle(t + i * T, rank_of(i, 0), (int)(ka[i] & 0xFFFFu));
      } else {
        tied_ranks(n_src, 0, settle);
      }
      int* mn = sh_min[round & 1];
      changed = wave_min(changed);
      ahead = wave_min(ahead);
      if (lane == 0 && changed != kNone) atomicMin(&mn[0], changed);
      if (lane == 0 && ahead != kNone) atomicMin(&mn[1], ahead);
      if (t == 0) sh_min[(round & 1) ^ 1][0] = sh_min[(round & 1) ^ 1][1] = kNone;
      __syncthreads();
      const int right = min(mn[0], mn[1]);                   // so many places are the queue's
      bool slow = false;
      if (round == kGuessRound) {                            // depths are not distinct: nothing follows from them yet
      } else if (right == kNone) {
        state = 1;
      } else if ((int)count[right + 1] == right) {
        state = 2;                                           // no other op has all its predecessors among them
      } else if ((round & (round < kGuessRound ? 15 : 7)) == (round < kGuessRound ? 15 : 7)) {
        // how many more rounds at the rate of the last sixteen or eight?
        const bool first = round < kGuessRound;
        slow = ((int)count[G + 1] - right) * (first ? 16 : 8) > (right - seen) * (first ? kSecondGuess : kWalkRounds + (G >> 5));
        seen = right;
        if (slow && !first) state = 3;
      }
      __syncthreads();
      if (__builtin_expect(slow && round < kGuessRound, 0)) {
        if (depths()) state = 2;
        round = kGuessRound - 1;
        seen = 0;
      }
    }
    if (state != 1) {
      if (t == 0) cost[c] = state == 2 ? INFINITY : __uint_as_float(kLeft);
      __syncthreads();
      continue;
    }
    // ---- the all-reduces by (place of the last predecessor, index), behind the ops
    unsigned n_of = 0;
    for (int i = 0; i < NPT; ++i) n_of += (is_op >> i) & 1u;
    const int lane_sum = wave_incl_scan((int)n_of);
    if (lane == 63) wsum[wave] = lane_sum;
    __syncthreads();
    int n_op = 0;
    for (int w = 0; w < kWaves; ++w) n_op += wsum[w];
    const int n_ar = G - n_op;
    __syncthreads();
    if (n_ar > 0) {
      sort(is_ar, 0, n_op);
      if (!ties) {
#pragma unroll
        for (int i = 0; i < NPT; ++i)
          if ((is_ar >> i) & 1u) ka[i] = (unsigned)rank_of(i, n_op) << 16 | (ka[i] & 0xFFFFu);
      } else {
        tied_ranks(0, n_op, [&](int v, int rank, int) { place[v] = (unsigned short)rank; });
#pragma unroll
        for (int i = 0; i < NPT; ++i)
          if ((is_ar >> i) & 1u) ka[i] = (unsigned)place[t + i * T] << 16 | (ka[i] & 0xFFFFu);
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NPT; ++i)
        if ((is_ar >> i) & 1u) {
          order[n_op + (ka[i] >> 16)] = (unsigned short)(t + i * T);
          place[t + i * T] = (unsigned short)ka[i];
        }
    }
    __syncthreads();
    // execution times and tensor sizes in that order
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const int v = t + i * T;
      if ((is_op >> i) & 1u) value[place[v] - 1] = op_time[n0 + v];
      if ((is_ar >> i) & 1u) value[n_op + (ka[i] >> 16)] = ar_size[n0 + v];
    }
    if (t == 0) sh_min[0][0] = sh_min[0][1] = kNone;
    __syncthreads();
    // ---- the times.  fp64 sums of fp32 values are exact, and so the same in any order, as long as no sum reaches 2^53
    // of the smallest value's last place: with the exponents' range known the clock at every op is a parallel scan,
    // and the serial chain is left for values that differ too much (or are infinite).
    double own = 0.0;                                        // the thread's NPT ops in the order
    {
      int lo = kNone, hi = kNone;                            // smallest exponent, 255 - largest
#pragma unroll
      for (int k = 0; k < NPT; ++k) {
        const int q = t * NPT + k;
        const float x = q < n_op ? value[q] : 0.f;
        const int ex = max((int)(__float_as_uint(x) >> 23 & 0xFFu), 1);
        if (x != 0.f) {
          lo = min(lo, ex);
          hi = min(hi, 255 - ex);
        }
        own += (double)x;
      }
      lo = wave_min(lo);
      hi = wave_min(hi);
      if (lane == 0 && lo != kNone) {
        atomicMin(&sh_min[0][0], lo);
        atomicMin(&sh_min[0][1], hi);
      }
    }
    double before = own;                                     // sum of the lanes up to this one
    for (int o = 1; o < 64; o <<= 1) {
      const double y = __shfl_up(before, o, 64);
      if (lane >= o) before += y;
    }
    if (lane == 63) sums[wave] = before;
    __syncthreads();
    const int lo = sh_min[0][0], hi = sh_min[0][1];
    const bool exact = lo == kNone || ((255 - hi) - lo + 24 + (32 - __clz(n_op)) <= 53 && hi > 0);
    double total = 0.0;
    for (int w = 0; w < kWaves; ++w) {
      const double x = sums[w];
      if (w < wave) before += x;
      total += x;
    }
    __syncthreads();
    if (exact) sums[t] = before - own;                       // the clock when the thread's first op begins
    __syncthreads();
    if (wave == 0) {
      double chan = 0.0;
      int e = 0;                                             // the next all-reduce; lane l holds number e0 + l
      int e0 = 0, by = 0;
      double run = 0.0;
      auto load_ar = [&]() {
        e0 = e;
        const bool ok = e0 + lane < n_ar;
        by = ok ? (int)place[order[n_op + e0 + lane]] : kNone;
        run = (double)ar_c * (double)(ok ? value[n_op + e0 + lane] : 0.f) + (double)ar_d;
      };
      // the channel's turn for n all-reduces from e on, produced at the lanes' r
      auto take = [&](double r, int n) {
        for (int k = e - e0; k < e - e0 + n; ++k) {
          const double rk = lane_of(r, k);
          chan = (rk > chan ? rk : chan) + lane_of(run, k);
        }
        e += n;
      };
      double dev = total;
      if (exact) {
        while (e < n_ar) {
          load_ar();
          const int b = by == kNone ? 0 : by;
          double r = sums[min(b / NPT, T - 1)];
          const int first = b / NPT < T ? b & ~(NPT - 1) : b - NPT;
#pragma unroll
          for (int k = 0; k < NPT; ++k) r += first + k < b ? (double)value[first + k] : 0.0;
          take(r, min(64, n_ar - e0));
        }
      } else {
        double* ends = sums;                                 // the clock after each of 64 ops
        double* runs = sums + 64;                            // their times
        auto produce = [&](int done, int first) {            // those produced by the first `done` ops
          while (e < n_ar) {
            if (e == e0 + 64) load_ar();
            const unsigned long long m = __ballot(by <= done) & (~0ull << (e - e0));
            if (m == 0) break;
            double r = 0.0;
            if (by <= done && by > 0 && e0 + lane >= e) r = ends[by - 1 - first];
            take(r, __popcll(m));
          }
        };
        if (n_ar > 0) load_ar();
        produce(0, 0);
        dev = 0.0;                                           // lane 0's is the clock
        for (int i0 = 0; i0 < n_op; i0 += 64) {
          runs[lane] = (double)(i0 + lane < n_op ? value[i0 + lane] : 0.f);
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
          if (lane == 0)
            for (int k = 0; k < 64; ++k) {
              dev += runs[k];
              ends[k] = dev;
            }
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
          produce(min(i0 + 64, n_op), i0);
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        }
      }
      if (lane == 0) cost[c] = (float)(dev > chan ? dev : chan);
    }
    __syncthreads();
  }
}

template <int T, int NPT>
hipError_t launch_order(const SimArgs& a, int fewest, bool last, hipStream_t s) {
  static bool attr_done = false;
  constexpr int bytes = OrderLds<T, NPT>::kBytes;
  if (!attr_done && bytes > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&simulate_order_kernel<T, NPT>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const int resident = a.n_cu * (2048 / T > 16 ? 16 : 2048 / T);
  hipLaunchKernelGGL((simulate_order_kernel<T, NPT>), dim3(a.n_cand < resident ? a.n_cand : resident), dim3(T), bytes, s,
                     a.node_off, a.out_rowptr, a.in_rowptr, a.in_col, a.op_time, a.ar_size, a.n_cand, a.ar_c, a.ar_d,
                     a.cost, fewest, (int)last, a.status);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------
// The walk of a module node by node, by one wave.  A chain of dependent accesses, about 800 cycles a node in LDS, so
// what counts is how many modules a CU walks at a time.
// ---------------------------------------------------------------------------------------------------
// LDS operations of a wave are carried out in issue order, so between a lane's write and another lane's later read only
// the compiler has to be kept from reordering; global memory needs the writes to have completed (there the workgroup
// is the one wave).
template <bool kLds>
__device__ __forceinline__ void sync_wave() {
  if (kLds) __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  else __syncthreads();
}

// base: the wave's working set, of sim_lds_bytes / sim_bytes of the module's G nodes and E edges
template <bool kLds>
__device__ __forceinline__ void walk_module(char* base, int n0, int G, int e0, int E, const int* __restrict__ out_rp,
                                            const int* __restrict__ out_ci, const int* __restrict__ in_rp,
                                            const float* __restrict__ op_time, const float* __restrict__ ar_size,
                                            float ar_c, float ar_d, float* __restrict__ cost) {
  typedef typename SimTypes<kLds>::dep_t dep_t;
  typedef typename SimTypes<kLds>::q_t q_t;
  constexpr int kAr = SimTypes<kLds>::kAr;
  const int lane = threadIdx.x & 63;
  double* ready = reinterpret_cast<double*>(base);
  float* val = reinterpret_cast<float*>(ready + G);      // execution time, or tensor size of an all-reduce
  dep_t* dep;
  q_t* qu;                 // every node is queued once: ops fill it from the front, all-reduces from the back
  int* rp;
  unsigned short* ci;
  if (kLds) {
    rp = reinterpret_cast<int*>(val + G);
    dep = reinterpret_cast<dep_t*>(rp + G + 1);
    qu = reinterpret_cast<q_t*>(dep + G);
    ci = reinterpret_cast<unsigned short*>(qu + G);
  } else {
    dep = reinterpret_cast<dep_t*>(val + G);
    qu = reinterpret_cast<q_t*>(dep + G);
    rp = reinterpret_cast<int*>(qu + G);
    ci = reinterpret_cast<unsigned short*>(rp + G + 1);
  }
  const double dc = (double)ar_c, dd = (double)ar_d;

  // ---- load the module
  for (int v = lane; v < G; v += 64) {
    const float x = ar_size[n0 + v];
    const bool ar = x >= 0.0f;
    ready[v] = 0.0;
    val[v] = ar ? x : op_time[n0 + v];
    dep[v] = (dep_t)((in_rp[n0 + v + 1] - in_rp[n0 + v]) | (ar ? kAr : 0));
    rp[v] = out_rp[n0 + v] - e0;
  }
  if (lane == 0) rp[G] = E;
  for (int k = lane; k < E; k += 64) ci[k] = (unsigned short)(out_ci[e0 + k] - n0);
  sync_wave<kLds>();

  // ---- sources, in ascending index, onto the two queues
  int qt = 0, at = 0;                   // entries queued so far (wave-uniform)
  for (int v0 = 0; v0 < G; v0 += 64) {
    const int v = v0 + lane;
    const int d = v < G ? dep[v] : 1;
    const bool src_op = d == 0, src_ar = d == kAr;
    const unsigned long long mo = __ballot(src_op), ma = __ballot(src_ar);
    const unsigned long long below = (1ull << lane) - 1ull;
    if (src_op) qu[qt + __popcll(mo & below)] = (q_t)v;
    if (src_ar) qu[G - 1 - (at + __popcll(ma & below))] = (q_t)v;
    qt += __popcll(mo);
    at += __popcll(ma);
  }
  sync_wave<kLds>();

  // ---- the walk
  int qh = 0, ah = 0, processed = 0;
  double dev = 0.0, chan = 0.0;
  while (ah < at || qh < qt) {
    int u;
    double done;
    if (ah < at) {                      // tensors already produced go on the channel first
      u = qu[G - 1 - ah++];
      const double r = ready[u];
      done = (r > chan ? r : chan) + (dc * (double)val[u] + dd);
      chan = done;
    } else {
      u = qu[qh++];
      const double r = ready[u];
      done = (r > dev ? r : dev) + (double)val[u];
      dev = done;
    }
    ++processed;
    const int s = rp[u], e = rp[u + 1];
    for (int k0 = s; k0 < e; k0 += 64) {
      const int k = k0 + lane;
      bool new_op = false, new_ar = false;
      int w = 0;
      if (k < e) {
        w = ci[k];
        if (done > ready[w]) ready[w] = done;
        const int d = (int)dep[w] - 1;
        dep[w] = (dep_t)d;
        new_op = d == 0;
        new_ar = d == kAr;
      }
      const unsigned long long mo = __ballot(new_op), ma = __ballot(new_ar);
      const unsigned long long below = (1ull << lane) - 1ull;
      if (new_op) qu[qt + __popcll(mo & below)] = (q_t)w;
      if (new_ar) qu[G - 1 - (at + __popcll(ma & below))] = (q_t)w;
      qt += __popcll(mo);
      at += __popcll(ma);
    }
    sync_wave<kLds>();                  // the releases are visible before the next node is taken
  }
  if (lane == 0) *cost = processed == G ? (float)(dev > chan ? dev : chan) : INFINITY;
  sync_wave<kLds>();
}

// The modules that simulate_order_kernel left and whose arrays fit LDS: a workgroup has a CU's LDS to itself and deals
// its modules to as many waves as working sets of their size class fit.  One launch for all classes: in the usual call,
// where nothing is left, a launch per class would cost as much as a small batch takes.  4096 modules in which ops wait
// for all-reduces, 2 waves on a CU whatever the size -> by classes: 1.6 k nodes 5.01 -> 2.77 ms, 0.7 k nodes
// 2.16 -> 0.94, 250 nodes 0.83 -> 0.27.
constexpr int kWalkClasses = 6;
constexpr int kWalkWaves = 10, kWalkThreads = 64 * kWalkWaves;
constexpr int kWalkList = 16;                                  // after the two counters: the modules of a class
constexpr int kWalkSlots = kWalkList + ((2 * kWalkThreads + 15) & ~15);
constexpr int kWalkLds = 160 * 1024 - 512;                     // less what __syncthreads_count takes
__host__ __device__ constexpr int walk_waves(int k) { return k == 0 ? 10 : k == 1 ? 6 : 6 - k; }      // 10, 6, 4, 3, 2, 1
__host__ __device__ constexpr int walk_slot(int k) { return (kWalkLds - kWalkSlots) / walk_waves(k) & ~15; }

__global__ __launch_bounds__(kWalkThreads) void simulate_walk_kernel(
    const int* __restrict__ node_off, const int* __restrict__ out_rp, const int* __restrict__ out_ci,
    const int* __restrict__ in_rp, const float* __restrict__ op_time, const float* __restrict__ ar_size, int C,
    float ar_c, float ar_d, float* __restrict__ cost, int lds_most, int last,
    unsigned long long* __restrict__ walked, int* status) {
  // lds_most: larger working sets are left to the kernel that follows; without one (last) such a module is an error
  if (call_failed(status)) return;
  int* ctr = reinterpret_cast<int*>(dc_sim_smem);
  unsigned short* list = reinterpret_cast<unsigned short*>(dc_sim_smem + kWalkList);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int mine = (C - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;      // modules blockIdx.x + k * gridDim.x
  for (int k0 = 0; k0 < mine; k0 += kWalkThreads) {
    int cls = kWalkClasses;
    const int c = blockIdx.x + (k0 + t) * gridDim.x;
    const bool left = k0 + t < mine && __float_as_uint(cost[c]) == kLeft;
    if (left) {
      const int n0 = node_off[c], G = node_off[c + 1] - n0;
      const size_t need = sim_lds_bytes(G, out_rp[n0 + G] - out_rp[n0]);
      if (need <= (size_t)lds_most)
        for (cls = 0; cls < kWalkClasses && need > (size_t)walk_slot(cls);) ++cls;
      if (cls == kWalkClasses && last) {                       // larger than any base graph of this context
        set_error(status, (int)DC_ERR_CAPACITY);
        cost[c] = INFINITY;
      }
    }
    const int n_left = __syncthreads_count(left);
    if (n_left == 0) continue;
    if (walked && t == 0) atomicAdd(walked, (unsigned long long)n_left);
#pragma unroll 1
    for (int k = 0; k < kWalkClasses; ++k) {
      if (t == 0) ctr[0] = ctr[1] = 0;
      __syncthreads();
      if (cls == k) list[atomicAdd(&ctr[0], 1)] = (unsigned short)t;
      __syncthreads();
      const int n = __builtin_amdgcn_readfirstlane(ctr[0]);
      if (wave < walk_waves(k)) {
        char* base = dc_sim_smem + kWalkSlots + __builtin_amdgcn_readfirstlane(wave) * walk_slot(k);
        for (;;) {
          int i = 0;
          if (lane == 0) i = atomicAdd(&ctr[1], 1);
          i = __builtin_amdgcn_readfirstlane(i);
          if (i >= n) break;
          const int cc = blockIdx.x + (k0 + __builtin_amdgcn_readfirstlane(list[i])) * gridDim.x;    // known to be one for the wave
          const int n0 = node_off[cc], G = node_off[cc + 1] - n0, e0 = out_rp[n0];
          walk_module<true>(base, n0, G, e0, out_rp[n0 + G] - e0, out_rp, out_ci, in_rp, op_time, ar_size, ar_c, ar_d,
                            cost + cc);
        }
      }
      __syncthreads();
    }
  }
}

// The modules that both kernels before it left, each in a slice of global memory.
__global__ __launch_bounds__(64) void simulate_walk_global_kernel(
    const int* __restrict__ node_off, const int* __restrict__ out_rp, const int* __restrict__ out_ci,
    const int* __restrict__ in_rp, const float* __restrict__ op_time, const float* __restrict__ ar_size, int C,
    float ar_c, float ar_d, float* __restrict__ cost, char* scratch, size_t stride, int* status) {
  if (status[0] != 0) return;
  for (int c = blockIdx.x; c < C; c += gridDim.x) {
    if (__float_as_uint(cost[c]) != kLeft) continue;
    const int n0 = node_off[c], G = node_off[c + 1] - n0;
    const int e0 = out_rp[n0], E = out_rp[n0 + G] - e0;
    if (sim_bytes(G, E) > stride) {                 // larger than any base graph of this context
      if (threadIdx.x == 0) {
        set_error(status, (int)DC_ERR_CAPACITY);
        cost[c] = INFINITY;
      }
      continue;
    }
    walk_module<false>(scratch + (size_t)blockIdx.x * stride, n0, G, e0, E, out_rp, out_ci, in_rp, op_time, ar_size, ar_c,
                       ar_d, cost + c);
  }
}

}  // namespace

size_t simulate_scratch_bytes(long long max_graph_nodes, long long max_graph_edges, int n_slices) {
  return sim_bytes(max_graph_nodes, max_graph_edges) * (size_t)n_slices;
}

hipError_t launch_simulate(const SimArgs& a, hipStream_t s) {
  if (a.n_cand <= 0) return hipSuccess;
  static bool attr_done = false;
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&simulate_walk_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kWalkLds);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  // classes of module size, up to what the largest module of the batch may need
  const int n = a.max_module_nodes;
  hipError_t e = launch_order<64, 4>(a, 0, n <= 256, s);
  if (e == hipSuccess && n > 256) e = launch_order<256, 8>(a, 257, n <= 2048, s);
  if (e == hipSuccess && n > 2048) e = launch_order<1024, 8>(a, 2049, n <= 8192, s);
  if (e == hipSuccess && n > 8192) e = launch_order<1024, 16>(a, 8193, true, s);
  if (e != hipSuccess) return e;
  // what it left
  hipLaunchKernelGGL(simulate_walk_kernel, dim3(a.n_cand < a.n_cu ? a.n_cand : a.n_cu), dim3(kWalkThreads), kWalkLds, s,
                     a.node_off, a.out_rowptr, a.out_col, a.in_rowptr, a.op_time, a.ar_size, a.n_cand, a.ar_c, a.ar_d,
                     a.cost, a.lds_bytes, a.n_slices == 0, a.walked, a.status);
  if (a.n_slices > 0)
    hipLaunchKernelGGL(simulate_walk_global_kernel, dim3(a.n_slices), dim3(64), 0, s, a.node_off, a.out_rowptr,
                       a.out_col, a.in_rowptr, a.op_time, a.ar_size, a.n_cand, a.ar_c, a.ar_d, a.cost, a.scratch,
                       a.scratch_stride, a.status);
  return hipGetLastError();
}

// ---- the simulator for callers that cannot allocate ------------------------------------------------
namespace {

constexpr int kStaticLdsBytes = 80 * 1024;              // modules up to this size are walked in LDS
constexpr int kStaticSlices = 64;                       // workgroups of the global-memory walk
constexpr size_t kStaticSliceBytes = 256 * 1024;        // working set of the largest module accepted
constexpr size_t kStaticHeaderBytes = 256;              // status words
// Device memory of the library itself: the status words and the slices of the global-memory walk.
// In host code this name only stands for the symbol; the address on each device comes from
// hipGetSymbolAddress (static_scratch below) and is what every kernel and launch receives.
static __device__ __align__(256) char dc_sim_static_scratch[kStaticHeaderBytes + kStaticSlices * kStaticSliceBytes];

constexpr int kMaxDevices = 64;
std::mutex g_static_mu;
char* g_static_ptr[kMaxDevices] = {};
int g_static_cus[kMaxDevices] = {};

// The scratch array's address on the current device (every device holds its own copy), looked up once.
hipError_t static_scratch(char** ptr, int* n_cu) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_static_mu);
  if (!g_static_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(dc_sim_static_scratch));
    if (e != hipSuccess) return e;
    int cus = 0;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    g_static_cus[dev] = cus > 0 ? cus : 1;
    g_static_ptr[dev] = static_cast<char*>(p);
  }
  *ptr = g_static_ptr[dev];
  *n_cu = g_static_cus[dev];
  return hipSuccess;
}

__global__ void export_status_kernel(const int* __restrict__ status, int* __restrict__ out) { out[0] = status[0]; }

thread_local const char* t_static_error = "";

}  // namespace
}  // namespace dc

extern "C" dc_status dc_simulate_static(const dc_batch* in, int32_t max_module_nodes, int32_t max_module_edges,
                                        const float* op_time, const float* ar_size, float ar_c, float ar_d, float* cost,
                                        int32_t* dev_status, void* stream) {
  using namespace dc;
  t_static_error = "";
  if (!in || in->n_cand < 0 || max_module_nodes < 0 || max_module_edges < 0) {
    t_static_error = "null batch or negative size";
    return DC_ERR_INVALID_ARG;
  }
  if (in->n_cand == 0) return DC_OK;
  if (!cost || !op_time || !ar_size || !in->node_off || !in->out_rowptr || !in->out_col || !in->in_rowptr || !in->in_col) {
    t_static_error = "null array";
    return DC_ERR_INVALID_ARG;
  }
  if (max_module_nodes >= 65536) {
    t_static_error = "a module has fewer than 65536 nodes";
    return DC_ERR_CAPACITY;
  }
  if (sim_bytes(max_module_nodes, max_module_edges) > kStaticSliceBytes) {
    t_static_error = "the largest module needs more than the 256 KiB working set this entry point holds: "
                     "24 bytes per node + 2 bytes per edge; use dc_simulate";
    return DC_ERR_CAPACITY;
  }
  char* scratch = nullptr;
  int n_cu = 0;
  hipError_t e = static_scratch(&scratch, &n_cu);
  if (e != hipSuccess) {
    t_static_error = hipGetErrorString(e);
    return DC_ERR_HIP;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  int* status = reinterpret_cast<int*>(scratch);
  hipLaunchKernelGGL(reset_status_kernel, dim3(1), dim3(1), 0, s, status);          // a fill kernel, not a memset
  launch_check_batch(in->node_off, in->n_cand, (long long)in->cap_nodes, (long long)in->cap_edges, in->out_rowptr,
                     in->out_col, in->in_rowptr, in->in_col, status, n_cu, s);
  SimArgs a;
  a.n_cand = in->n_cand;
  a.node_off = in->node_off;
  a.out_rowptr = in->out_rowptr;
  a.out_col = in->out_col;
  a.in_rowptr = in->in_rowptr;
  a.in_col = in->in_col;
  a.max_module_nodes = max_module_nodes;
  a.op_time = op_time;
  a.ar_size = ar_size;
  a.ar_c = ar_c;
  a.ar_d = ar_d;
  a.cost = cost;
  a.lds_bytes = kStaticLdsBytes;
  a.scratch = scratch + kStaticHeaderBytes;
  a.scratch_stride = kStaticSliceBytes;
  a.n_slices = kStaticSlices;
  a.n_cu = n_cu;
  a.walked = nullptr;
  a.status = status;
  e = launch_simulate(a, s);
  if (e == hipSuccess && dev_status) {
    hipLaunchKernelGGL(export_status_kernel, dim3(1), dim3(1), 0, s, status, dev_status);
    e = hipGetLastError();
  }
  if (e != hipSuccess) {
    t_static_error = hipGetErrorString(e);
    return DC_ERR_HIP;
  }
  return DC_OK;
}

extern "C" const char* dc_simulate_static_error(void) { return dc::t_static_error; }
