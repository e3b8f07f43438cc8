// Backtracking search over fusion strategies (Alg. 1, Sec. 4) on top of the batched cost model.
//
// A strategy is a labelling of the base nodes; H_in is the all-singleton labelling.  Per step
// up to `parents` entries leave the priority queue (ascending cost, then age); every parent
// gets one child per optimisation method, drawn on the device by mutate_kernel (RandomApply:
// n = Random(0, beta) applications of the method); the children are costed in one
// dc_cost_candidates call and then handled in order on the host: a valid child (finite cost)
// replaces H_opt when cheaper, which restarts the counter of unchanged evaluations, and is
// enqueued when Cost(H') <= alpha * Cost(H_opt).  The search ends when the queue is empty, the
// counter reaches its limit (checked between steps) or max_steps is reached.  parents = 1 is
// the loop as printed.
//
// Methods (Sec. 4, (i) and (iii); (ii) duplicates an op, which no labelling of the node set
// expresses):  op fusion, one application, in one of two forms.  DC_DRAW_DEPENDENCY: a dependency
// u -> v between two computation ops of the base module is drawn uniformly; if its ends lie in
// different groups, the group of u joins the group of v.  DC_DRAW_OP (the paper's wording): a
// computation op of the current module is drawn uniformly (the groups of the labelling, in the
// order of their smallest member), then one of its predecessor ops in the current module
// uniformly (the groups with a dependency into it, same order), and the predecessor joins the
// op; an op without predecessors leaves the module as it is; the low half of the 64-bit draw
// picks the op, the high half the predecessor.  Tensor fusion, one application: an all-reduce node a and a side are
// drawn uniformly; the nearest bucket on that side in production order, if there is one,
// joins the bucket of a.  Validity is what the cost reports: a cyclic module costs +infinity.
//
// Draws: key = mix(seed ^ mix(step * 2^32 + child)), draw d = mix(key + d * 0xD1342543DE82EF95)
// with mix = splitmix64's output function; draw 0 gives n, draws 1.. the applications.
#include <math.h>
#include <string.h>

#include <set>
#include <tuple>
#include <vector>

#include "common.h"

namespace dc {
namespace {

constexpr int kMutateThreads = 512;
constexpr int kMutateLdsLimit = 160 * 1024 - 2048;   // dynamic LDS of mutate_kernel next to its static arrays

__host__ __device__ inline unsigned long long mix64(unsigned long long x) {
  unsigned long long z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

extern __shared__ __attribute__((aligned(16))) unsigned short dc_search_lab[];

// The k-th (from 0) set bit of bits[0 .. words), or -1 if there are none; `pick` is called with their number and
// returns k.  Every wave of the workgroup does this by itself and gets the same answer: no barrier.
template <typename Pick>
__device__ __forceinline__ int kth_bit(const unsigned* bits, int words, Pick pick) {
  const int lane = threadIdx.x & 63;
  const int per = (words + 63) >> 6, lo = min(lane * per, words), hi = min(lo + per, words);
  int c = 0;
  for (int w = lo; w < hi; ++w) c += __popc(bits[w]);
  const int upto = wave_incl_scan(c);
  const int total = __builtin_amdgcn_readlane(upto, 63);
  if (total == 0) return -1;
  int k = pick(total);
  const int l = __ffsll((unsigned long long)__ballot(upto > k)) - 1;      // the lane that holds it
  k -= __builtin_amdgcn_readlane(upto - c, l);
  int w = l * per;
  unsigned x = bits[w];
  for (int n = __popc(x); k >= n; n = __popc(x)) {
    k -= n;
    x = bits[++w];
  }
  // lane i: is bit i the one with k set bits below it
  const bool me = lane < 32 && ((x >> (lane & 31)) & 1u) && __popc(x & ((1u << (lane & 31)) - 1u)) == k;
  return w * 32 + __ffsll((unsigned long long)__ballot(me)) - 1;
}

// One workgroup per child: child j descends from parent j / 2 by method j % 2.  Labels in LDS as 16-bit values.
// op_draw != 0 takes the paper's draw for op fusion and needs, behind the labels, the smallest op per label (4 N
// bytes), a bit per node that heads its group and two times a bit per node for the marks, and, as far as edges_in_lds
// says, the dependencies (4 bytes each).  Heads and smallest ops follow the merges: only the first application reads
// all labels for them.  What bounds it: up to beta applications after each other, each the scan of the dependencies
// and of the labels between two barriers; the selections are wave-wide scans of bitmaps that every wave does for
// itself.  Measured, 16 children of a 729-node module, five applications on average: 117 us when one thread added up
// the counts of a selection and every application found heads and marks anew, 17 us now.
__global__ __launch_bounds__(kMutateThreads) void mutate_kernel(const int* __restrict__ pool, const int* __restrict__ parent_slot,
                                                      int N, int n_edges, const unsigned* __restrict__ edges, int n_ar,
                                                      const int* __restrict__ ar_nodes, int n_op,
                                                      const int* __restrict__ op_nodes, int op_draw, int edges_in_lds,
                                                      unsigned long long seed, unsigned long long step, int beta,
                                                      int* __restrict__ children) {
  unsigned short* lab = dc_search_lab;
  int* first = reinterpret_cast<int*>(lab + ((N + 1) & ~1));
  const int words = (N + 31) >> 5;
  unsigned* head = reinterpret_cast<unsigned*>(first + N);
  unsigned* mark = head + words;                             // [2][words]
  unsigned* edge_lds = mark + 2 * words;
  const int j = blockIdx.x, t = threadIdx.x, T = blockDim.x, lane = t & 63;
  const int method = j & 1;
  const int* src = pool + (size_t)parent_slot[j >> 1] * N;
  const unsigned long long key = mix64(seed ^ mix64((step << 32) + (unsigned long long)j));
  const int n = (int)(mix64(key) % (unsigned long long)(beta + 1));
  const bool paper = method == 0 && op_draw != 0;
  for (int v = t; v < N; v += T) lab[v] = (unsigned short)src[v];
  if (paper && n > 0) {
    for (int v = t; v < N; v += T) first[v] = 0x7FFFFFFF;
    for (int w = t; w < 3 * words; w += T) head[w] = 0;      // and the marks behind it
    if (edges_in_lds)
      for (int e = t; e < n_edges; e += T) edge_lds[e] = edges[e];
    __syncthreads();
    for (int q = t; q < n_op; q += T) atomicMin(&first[lab[op_nodes[q]]], op_nodes[q]);
    __syncthreads();
    for (int q = t; q < n_op; q += T) {
      const int v = op_nodes[q];
      if (first[lab[v]] == v) atomicOr(&head[v >> 5], 1u << (v & 31));
    }
  }
  __syncthreads();
  const unsigned* ed = edges_in_lds ? edge_lds : edges;
  for (int i = 0; i < n; ++i) {
    const unsigned long long r = mix64(key + (unsigned long long)(1 + i) * 0xD1342543DE82EF95ull);
    int from = -1, to = -1, gone = -1, stays = -1;           // heads of the two groups, for the paper's draw
    if (paper) {
      const int qo = kth_bit(head, words, [&](int total) { return (int)((unsigned)r % (unsigned)total); });
      if (qo >= 0) {
        const int op = lab[qo];
        unsigned* mk = mark + (i & 1) * words;
        for (int e = t; e < n_edges; e += T) {
          const unsigned x = ed[e];
          const int lu = lab[x & 0xFFFFu];
          if (lab[x >> 16] == op && lu != op) {
            const int h = first[lu];
            atomicOr(&mk[h >> 5], 1u << (h & 31));
          }
        }
        __syncthreads();
        const int qp = kth_bit(mk, words, [&](int total) { return (int)((unsigned)(r >> 32) % (unsigned)total); });
        if (qp >= 0) {
          from = lab[qp];
          to = op;
          gone = max(qo, qp);
          stays = min(qo, qp);
        }
        for (int w = t; w < words; w += T) mark[((i & 1) ^ 1) * words + w] = 0;      // the next application's
      }
    } else if (method == 0) {
      if (n_edges > 0) {
        const unsigned x = ed[r % (unsigned long long)n_edges];
        from = lab[x & 0xFFFFu];
        to = lab[x >> 16];
      }
    } else if (n_ar > 0) {
      const int pa = (int)(r % (unsigned long long)n_ar);
      const int side = ((r >> 32) & 1ull) ? 1 : -1;
      const int la = lab[ar_nodes[pa]];
      // the nearest tensor on that side with another label, 64 places at a time
      for (int p0 = pa + side; p0 >= 0 && p0 < n_ar && from < 0; p0 += 64 * side) {
        const int p = p0 + lane * side;
        const int l = p >= 0 && p < n_ar ? (int)lab[ar_nodes[p]] : la;
        const unsigned long long m = __ballot(l != la);
        if (m) {
          from = __builtin_amdgcn_readlane(l, __ffsll(m) - 1);
          to = la;
        }
      }
    }
    __syncthreads();                                         // everyone has read the labels and the heads
    if (from >= 0 && from != to) {
      for (int v = t; v < N; v += T)
        if (lab[v] == from) lab[v] = (unsigned short)to;
      if (paper && t == 0) {
        first[to] = stays;
        head[gone >> 5] &= ~(1u << (gone & 31));
      }
    }
    __syncthreads();
  }
  int* dst = children + (size_t)j * N;
  for (int v = t; v < N; v += T) dst[v] = lab[v];
}

// Copies the children that were kept into their pool slots: pair i = (child, slot).
__global__ __launch_bounds__(256) void keep_kernel(const int* __restrict__ children, int* __restrict__ pool, int N,
                                                    const int* __restrict__ pairs) {
  const int* src = children + (size_t)pairs[2 * blockIdx.x] * N;
  int* dst = pool + (size_t)pairs[2 * blockIdx.x + 1] * N;
  for (int v = threadIdx.x; v < N; v += blockDim.x) dst[v] = src[v];
}

__global__ void iota_kernel(int* p, int n, int mul) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = i * mul;
}
__global__ void fill_kernel(int* p, int n, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

struct DevMem {
  std::vector<void*> ptrs;
  void* pinned = nullptr;
  ~DevMem() {
    for (void* p : ptrs) (void)hipFree(p);
    if (pinned) (void)hipHostFree(pinned);
  }
  template <typename T>
  T* take(size_t n, hipError_t* e) {
    void* p = nullptr;
    if (*e == hipSuccess) *e = hipMalloc(&p, (n ? n : 1) * sizeof(T));
    if (p) ptrs.push_back(p);
    return static_cast<T*>(p);
  }
};

}  // namespace

dc_status run_search(dc_ctx* ctx, const SearchView& g, int32_t graph, const dc_search_params& p, int32_t* labels_opt,
                     dc_search_result* res, hipStream_t s) {
  const int N = g.n, P = p.parents, C = 2 * P;
  // op-op dependencies in CSR order and all-reduce nodes in production order, built on the host
  std::vector<int> rp(N + 1), ci(g.e > 0 ? g.e : 1);
  std::vector<float> ar(N > 0 ? N : 1);
  hipError_t e = hipMemcpyAsync(rp.data(), g.rowptr, (N + 1) * sizeof(int), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess && g.e > 0) e = hipMemcpyAsync(ci.data(), g.col, (size_t)g.e * sizeof(int), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess && N > 0) e = hipMemcpyAsync(ar.data(), g.ar_size, (size_t)N * sizeof(float), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return DC_ERR_HIP;
  std::vector<int> arn, opn;
  std::vector<unsigned> edges;               // source | target << 16
  for (int u = 0; u < N; ++u) {
    if (ar[u] >= 0.0f) {
      arn.push_back(u);
      continue;
    }
    opn.push_back(u);
    for (int k = rp[u]; k < rp[u + 1]; ++k)
      if (ar[ci[k]] < 0.0f) edges.push_back((unsigned)u | (unsigned)ci[k] << 16);
  }
  const int slots = p.max_queue + C + 4;
  DevMem mem;
  unsigned* d_edges = mem.take<unsigned>(edges.size(), &e);
  int* d_arn = mem.take<int>(arn.size(), &e);
  int* d_opn = mem.take<int>(opn.size(), &e);
  int* pool = mem.take<int>((size_t)slots * N, &e);
  int* children = mem.take<int>((size_t)C * N, &e);
  int* cand_graph = mem.take<int>(C, &e);
  int* cand_off = mem.take<int>(C + 1, &e);
  float* d_cost = mem.take<float>(C, &e);
  if (e == hipSuccess)
    e = hipHostMalloc(&mem.pinned, (size_t)C * sizeof(float) + ((size_t)P + 2 * (size_t)(C + 1)) * sizeof(int),
                      hipHostMallocDefault);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return e == hipErrorOutOfMemory ? DC_ERR_OOM : DC_ERR_HIP;
  }
  // pinned memory: the kernels read the few parents and pairs of a step where the host wrote them, without copies
  float* h_cost = static_cast<float*>(mem.pinned);
  int* h_parent = reinterpret_cast<int*>(h_cost + C);
  int* h_pairs = h_parent + P;
  if (!edges.empty()) e = hipMemcpyAsync(d_edges, edges.data(), edges.size() * sizeof(unsigned), hipMemcpyHostToDevice, s);
  if (e == hipSuccess && !arn.empty()) e = hipMemcpyAsync(d_arn, arn.data(), arn.size() * sizeof(int), hipMemcpyHostToDevice, s);
  if (e == hipSuccess && !opn.empty()) e = hipMemcpyAsync(d_opn, opn.data(), opn.size() * sizeof(int), hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return DC_ERR_HIP;
  const int op_draw = p.op_draw == DC_DRAW_OP ? 1 : 0;
  // labels as 16-bit values; the paper's op draw also keeps a 32-bit smallest member per label, three bits per node
  // and, where they fit beside these, the dependencies
  size_t lds = (size_t)((N + 1) & ~1) * sizeof(unsigned short);
  if (op_draw) lds += (size_t)N * 4 + 3 * (((size_t)N + 31) / 32) * 4;
  if (lds > (size_t)kMutateLdsLimit) return DC_ERR_UNSUPPORTED;
  const int edges_in_lds = op_draw && lds + edges.size() * 4 <= (size_t)kMutateLdsLimit;
  if (edges_in_lds) lds += edges.size() * 4;
  if (lds > 48 * 1024) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&mutate_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds);
    if (e != hipSuccess) return DC_ERR_HIP;
  }
  hipLaunchKernelGGL(fill_kernel, dim3((C + 255) / 256), dim3(256), 0, s, cand_graph, C, graph);
  hipLaunchKernelGGL(iota_kernel, dim3((C + 1 + 255) / 256), dim3(256), 0, s, cand_off, C + 1, N);
  // slot 0: H_opt; slot 1: H_in (identity labels)
  std::vector<int> free_slots;
  for (int i = slots - 1; i >= 2; --i) free_slots.push_back(i);
  hipLaunchKernelGGL(iota_kernel, dim3((N + 255) / 256), dim3(256), 0, s, pool, N, 1);
  hipLaunchKernelGGL(iota_kernel, dim3((N + 255) / 256), dim3(256), 0, s, pool + (size_t)N, N, 1);
  auto cost_of = [&](const int* labels, int n) -> dc_status {
    dc_status st = dc_cost_candidates(ctx, n, cand_graph, cand_off, labels, p.ar_c, p.ar_d, d_cost, s);
    if (st != DC_OK) return st;
    if (hipMemcpyAsync(h_cost, d_cost, (size_t)n * sizeof(float), hipMemcpyDeviceToHost, s) != hipSuccess) return DC_ERR_HIP;
    return dc_check(ctx, s);                 // synchronises the stream
  };
  dc_status st = cost_of(pool + (size_t)N, 1);
  if (st != DC_OK) return st;
  const float cost_in = h_cost[0];
  float cost_opt = cost_in;
  typedef std::tuple<float, long long, int> Entry;   // cost, age, slot
  std::set<Entry> queue;
  queue.insert(Entry(cost_in, 0, 1));
  long long next_id = 1, step = 0, evaluated = 0, valid = 0, enqueued = 0, improved = 0;
  int unchanged = 0;
  std::vector<int> used;
  while (!queue.empty() && unchanged < p.max_unchanged && step < p.max_steps) {
    used.clear();
    while ((int)used.size() < P && !queue.empty()) {
      used.push_back(std::get<2>(*queue.begin()));
      queue.erase(queue.begin());
    }
    const int np = (int)used.size(), nc = 2 * np;
    for (int i = 0; i < np; ++i) h_parent[i] = used[i];
    hipLaunchKernelGGL(mutate_kernel, dim3(nc), dim3(kMutateThreads), lds, s, pool, h_parent, N, (int)edges.size(), d_edges,
                       (int)arn.size(), d_arn, (int)opn.size(), d_opn, op_draw, edges_in_lds, (unsigned long long)p.seed,
                       (unsigned long long)step, p.beta, children);
    if (hipGetLastError() != hipSuccess) return DC_ERR_HIP;
    st = cost_of(children, nc);
    if (st != DC_OK) return st;
    // decisions first, on the host; the label vectors that are kept move afterwards in one launch.
    // A slot that is given up within the step (queue full) may be handed out again: its earlier
    // pair is then dropped, so that no two pairs write one slot.
    int n_pairs = 0, best_child = -1;
    for (int j = 0; j < nc; ++j) {
      const float c = h_cost[j];
      ++evaluated;
      if (!isfinite(c)) continue;
      ++valid;
      if (c < cost_opt) {
        cost_opt = c;
        ++improved;
        unchanged = 0;
        best_child = j;
      } else {
        ++unchanged;
      }
      if ((double)c <= (double)p.alpha * (double)cost_opt) {
        if (free_slots.empty()) {            // the queue is full: its most expensive entry makes room
          if (queue.empty()) return DC_ERR_CAPACITY;
          auto last = std::prev(queue.end());
          const int gone = std::get<2>(*last);
          for (int i = 0; i < n_pairs; ++i)
            if (h_pairs[2 * i + 1] == gone) {
              h_pairs[2 * i] = h_pairs[2 * (n_pairs - 1)];
              h_pairs[2 * i + 1] = h_pairs[2 * (n_pairs - 1) + 1];
              --n_pairs;
              break;
            }
          free_slots.push_back(gone);
          queue.erase(last);
        }
        const int slot = free_slots.back();
        free_slots.pop_back();
        h_pairs[2 * n_pairs] = j;
        h_pairs[2 * n_pairs + 1] = slot;
        ++n_pairs;
        queue.insert(Entry(c, next_id++, slot));
        ++enqueued;
      }
    }
    if (best_child >= 0) {                   // slot 0 holds H_opt
      h_pairs[2 * n_pairs] = best_child;
      h_pairs[2 * n_pairs + 1] = 0;
      ++n_pairs;
    }
    if (n_pairs > 0) {
      hipLaunchKernelGGL(keep_kernel, dim3(n_pairs), dim3(256), 0, s, children, pool, N, h_pairs);
      if (hipGetLastError() != hipSuccess) return DC_ERR_HIP;
      // h_pairs is reused next step, which synchronises on its costs before it writes it again
    }
    for (int i = 0; i < np; ++i) free_slots.push_back(used[i]);
    while ((long long)queue.size() > (long long)p.max_queue) {
      auto last = std::prev(queue.end());
      free_slots.push_back(std::get<2>(*last));
      queue.erase(last);
    }
    ++step;
  }
  if (labels_opt) {
    if (hipMemcpyAsync(labels_opt, pool, (size_t)N * sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess) return DC_ERR_HIP;
  }
  if (hipStreamSynchronize(s) != hipSuccess) return DC_ERR_HIP;
  if (res) {
    res->cost_in = cost_in;
    res->cost_opt = cost_opt;
    res->steps = step;
    res->evaluated = evaluated;
    res->valid = valid;
    res->enqueued = enqueued;
    res->improved = improved;
    res->queued = (int64_t)queue.size();
    res->unchanged = unchanged;
  }
  return DC_OK;
}

}  // namespace dc
