// GPU scheduler for dynamic batching (Section 2 of the paper, the greedy
// scheduling algorithm), gfx950.
//
//   validate   CSR structure, op ids, arity, child range / same graph, inputs
//   depth      one workgroup per graph walks it bottom-up along the reverse edges in LDS: the thread that closes a
//              node's last child goes on with that node, at depth 1 + max(child depths) (the zero state -1 and
//              leaf-table rows are depth-0 constants).  Nodes never closed mean a cycle.
//   sort       stable LSD radix sort (10-bit digits) of the node ids by the key (depth - 1) * num_ops + op: ties stay in
//              node-id order.  A pass is a count and a scatter over tiles of 2,048 items (a column scan between them
//              only where there are many tiles)
//   emit       two passes over the sorted tiles: sums per tile, then every index: group table, level_ptr, child_pos (pool
//              rows of every edge), input_idx, root rows, the rows of every op in (op, row) order for the deferred
//              weight gradients, and the rows that read the leaf table, which one more sort lists by (op, leaf-table row)
// All results are integers and bit-exact by construction.  Everything runs on
// the stream without a host round trip until one read-back at the end: arrays
// are sized by N (levels and groups never outnumber nodes), the radix passes
// the actual depth needs are decided on the device, and every kernel after
// validation that uses a value as an index returns at once when the error word
// is set (the scans do not look at it: they add up arrays of fixed length).

#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstring>

#include "common.h"
#include "internal.h"
#include "pool.h"

namespace fold {

namespace {

constexpr unsigned long long kNoErr = ~0ull;
constexpr int kTooDeep = 0x7fffffff;  // error-word node of "depth * num_ops too large for the sort keys"
constexpr long long kMaxKeys = 1LL << 30;
constexpr int kBlock = 256;
constexpr int kMaxOps = 256;  // the op table travels as a kernel argument
constexpr int kScanItems = 8;        // items per thread in device-wide scans
constexpr int kScanTile = kBlock * kScanItems;
constexpr int kTileThreads = 512, kTileItems = 4, kTile = kTileThreads * kTileItems;  // items of a sort or emit tile
constexpr int kDigitBits = 10, kDigits = 1 << kDigitBits;
// Up to this many tiles every tile adds up its predecessors' digit counts itself (32 x 4 KB from the L2, about 3 us);
// above, a column scan does it once in a launch of its own (1,000 tiles: 4 MB, which every tile would read)
constexpr int kSelfTiles = 32;

struct OpTable {
  int n;
  unsigned char bits[kMaxOps];  // arity, and 4 where the operation reads the leaf table
  __host__ __device__ int arity(int op) const { return bits[op] & 3; }
  __host__ __device__ int has_input(int op) const { return bits[op] >> 2; }
};

// error word: ((node + 1) << 8) | (-code); structural errors use node + 1 = 0.  atomicMin keeps the
// lowest node with an error and, within it, the first check in the order op, arity, child, input.  Cycles have a word
// of their own: a graph's counts only where no check of any graph failed.
__device__ __forceinline__ void report(unsigned long long* err, int node_plus_1, int code) {
  unsigned long long w = ((unsigned long long)(unsigned)node_plus_1 << 8) | (unsigned long long)(-code);
  atomicMin(err, w);
}

// ---------------------------------------------------------------- block scan helpers

// exclusive scan of one int per thread over a workgroup of NT threads; returns the prefix, *total = sum
template <int NT>
__device__ int block_exscan(int x, int* total) {
  __shared__ int wsum[NT / kWave];
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  int v = x;
  for (int d = 1; d < kWave; d <<= 1) {
    int y = __shfl_up(v, d, kWave);
    if (lane >= d) v += y;
  }
  if (lane == kWave - 1) wsum[w] = v;
  __syncthreads();
  int pre = 0, tot = 0;
  for (int i = 0; i < NT / kWave; ++i) {
    int s = wsum[i];
    if (i < w) pre += s;
    tot += s;
  }
  __syncthreads();
  *total = tot;
  return pre + v - x;
}

// sum of one int per thread over a workgroup of NT threads, in every thread
template <int NT>
__device__ int block_sum(int x) {
  int total;
  (void)block_exscan<NT>(x, &total);
  return total;
}

// ---------------------------------------------------------------- validation

__global__ void k_check_struct(const int* gp, int G, const int* cp, int N, int E, unsigned long long* err) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) {
    if (gp[0] != 0 || gp[G] != N || cp[0] != 0 || cp[N] != E) report(err, 0, FOLD_E_INVALID);
  }
  if (i < G) {
    int a = gp[i], b = gp[i + 1];
    if (a < 0 || b > N || a > b) report(err, 0, FOLD_E_INVALID);
  }
  if (i < N) {
    int a = cp[i], b = cp[i + 1];
    if (a < 0 || b > E || a > b) report(err, 0, FOLD_E_INVALID);
  }
}

__global__ void k_node_graph(const int* gp, int* node_graph, const unsigned long long* err) {
  if (*err != kNoErr) return;
  const int g = blockIdx.x;
  for (int v = gp[g] + threadIdx.x; v < gp[g + 1]; v += blockDim.x) node_graph[v] = g;
}

// ---------------------------------------------------------------- depth (one workgroup per graph)

// Depths of one graph, bottom-up over its reverse edges: the node that delivers a parent's last child finishes that
// parent and goes on with it, so a chain runs in one lane from step to step with no barrier and no queue.  What
// bounds it is the chain of dependent LDS accesses per step (the parent link, then one returning atomic); a
// level-synchronous frontier paid two barriers, a queue and generic-address atomics per level instead (4,096 graphs,
// 2.0 M nodes, 511-node chains among them: 700 us, now 182; 1,024 sentiment trees: 101 us, now 26; 512 LSTM chains of
// up to 100 steps under reduce trees: 75 us, now 64).
// Parents of a node are a linked list of its edges; a node with one parent keeps that parent's number itself.  A lane
// that finishes several parents at once goes on with the lowest (the nearest one up a chain, where nodes are numbered
// children first) and puts the others on a list, which the next round takes.
//
// Where the links live: Lds, or Glob for a graph that does not fit (the same steps on 32-bit indices in scratch
// memory; what atomics write is read through atomics there, past the first-level cache).  ARITY2: at most two
// children, and one atomic both counts a child in and hands over its depth (count in the top byte, the depths summed
// below it: the second child reads the first one's); otherwise a maximum and a count.
//
// Threads of a workgroup, by the nodes of an average graph.  A walk is one lane's chain, but linking and checking go node
// by node: a graph of 100,000 nodes takes 3,434 us with 128 threads, 1,921 with 256, 694 with 1,024 (8 of 10,000: 408, 275,
// 156).  Graphs of a few hundred nodes fit the LDS and take the same with any (4,096 of 511: 327, 320, 335), and many tiny
// ones are bound by starting waves (100,000 of one node: 214, 254, 810).  A large graph among small ones gets 256 (20,000
// nodes among 1,000 graphs of 20: within 3 % of 1,024, the chains take the time).
inline int graph_threads(long long N, int G) {
  const long long mean = N / std::max(G, 1);
  return mean >= 1024 ? 1024 : (mean >= 16 ? 256 : 128);
}

// Parent edges of v, once all are linked; a single one is replaced by its parent's number.
template <class L>
__device__ __forceinline__ int close_node(const L& g, int v) {
  int k = 0, p = 0;
  unsigned nx;
  for (unsigned j = g.get_head(v); j != L::kNone; j = nx) p = g.get_edge(j, nx), ++k;
  if (k == 1) g.set_head(v, L::kSingle | (unsigned)p);
  return k;
}

template <bool ARITY2>
struct LdsLinks {
  static constexpr unsigned kNone = 0xffffu, kSingle = 0x80000000u;  // kNone has no kSingle bit
  static constexpr int kNodeBytes = ARITY2 ? 10 : 14, kEdgeBytes = 4;
  uint32_t *state, *depth, *head, *edge;
  uint16_t* list;
  __device__ __forceinline__ LdsLinks() {}
  __device__ __forceinline__ LdsLinks(char* at, int n, int e) {
    state = reinterpret_cast<uint32_t*>(at);
    head = state + n;
    depth = head + n;
    edge = ARITY2 ? depth : depth + n;
    list = reinterpret_cast<uint16_t*>(edge + e);
  }
  // edge j comes from parent p, the node's next one is nx
  __device__ __forceinline__ void set_edge(int j, int p, unsigned nx) const { edge[j] = (unsigned)p | nx << 16; }
  __device__ __forceinline__ int get_edge(unsigned j, unsigned& nx) const {
    const uint32_t x = edge[j];
    nx = x >> 16;
    return (int)(x & 0xffffu);
  }
  __device__ __forceinline__ unsigned get_head(int v) const { return head[v]; }
  __device__ __forceinline__ void set_head(int v, unsigned h) const { head[v] = h; }
  __device__ __forceinline__ unsigned link(int c, int j) const { return atomicExch(&head[c], (unsigned)j); }
  __device__ __forceinline__ void wait_for(int v, int children) const {
    if constexpr (ARITY2) {
      state[v] = (unsigned)(2 - children) << 24;
    } else {
      state[v] = (unsigned)children;
      depth[v] = 0;
    }
  }
  __device__ __forceinline__ void set_depth(int v, int d) const {
    if constexpr (ARITY2) state[v] = (unsigned)d;
    else depth[v] = (unsigned)d;
  }
  __device__ __forceinline__ int get_depth(int v) const { return (int)(ARITY2 ? state[v] : depth[v]); }
  __device__ __forceinline__ int close(int v) const { return close_node(*this, v); }
  // a child one step below depth d reports to p; true when it was the last one, with p's depth
  __device__ __forceinline__ bool arrive(int p, int d, int& dp) const {
    if constexpr (ARITY2) {
      const uint32_t old = atomicAdd(&state[p], (1u << 24) + (unsigned)d);
      dp = max((int)(old & 0xffffffu), d);
      return (old >> 24) == 1;
    } else {
      atomicMax(&depth[p], (unsigned)d);
      if (atomicSub(&state[p], 1u) != 1u) return false;
      dp = (int)__hip_atomic_load(&depth[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      return true;
    }
  }
};

template <bool ARITY2>
struct GlobLinks {
  static constexpr unsigned kNone = 0x7fffffffu, kSingle = 0x80000000u;
  static constexpr int kNodeInts = 4, kEdgeInts = 2;  // of scratch
  unsigned long long* state;  // ARITY2: count and sum of depths; else the count (low) and the depth (high word)
  int *head, *list, *next, *from;
  __device__ __forceinline__ GlobLinks(int* at, int n, int e) {
    state = reinterpret_cast<unsigned long long*>(at);
    head = at + 2 * (size_t)n;
    list = head + n;
    next = list + n;
    from = next + e;
  }
  template <class U>
  __device__ __forceinline__ static U now(const U* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ unsigned* word(int v, int k) const { return reinterpret_cast<unsigned*>(state + v) + k; }
  __device__ __forceinline__ void set_edge(int j, int p, unsigned nx) const {
    from[j] = p;
    next[j] = (int)nx;
  }
  __device__ __forceinline__ int get_edge(unsigned j, unsigned& nx) const {
    nx = (unsigned)next[j];
    return from[j];
  }
  __device__ __forceinline__ unsigned get_head(int v) const { return (unsigned)now(head + v); }
  __device__ __forceinline__ void set_head(int v, unsigned h) const { head[v] = (int)h; }
  __device__ __forceinline__ unsigned link(int c, int j) const { return (unsigned)atomicExch(&head[c], j); }
  __device__ __forceinline__ void wait_for(int v, int children) const {
    state[v] = ARITY2 ? (unsigned long long)(2 - children) << 56 : (unsigned long long)children;
  }
  __device__ __forceinline__ void set_depth(int v, int d) const {
    if constexpr (ARITY2) state[v] = (unsigned long long)d;
    else *word(v, 1) = (unsigned)d;
  }
  __device__ __forceinline__ int get_depth(int v) const { return (int)(ARITY2 ? now(state + v) : now(word(v, 1))); }
  __device__ __forceinline__ bool arrive(int p, int d, int& dp) const {
    if constexpr (ARITY2) {
      const unsigned long long old = atomicAdd(&state[p], (1ull << 56) + (unsigned)d);
      dp = max((int)(old & 0xffffffffull), d);
      return (old >> 56) == 1;
    } else {
      atomicMax(word(p, 1), (unsigned)d);
      __threadfence();  // the maximum is in before the count
      if (atomicSub(word(p, 0), 1u) != 1u) return false;
      dp = (int)now(word(p, 1));
      return true;
    }
  }
};

// what the workgroup of one graph shares beside the links
struct GraphShared {
  int tail, done, deepest, parents, bad;
};

struct GraphArgs {
  const int *gp, *cp, *ci;
  int *depth, *indeg, *scratch;
  unsigned long long *err, *cycle;
  int* meta;  // [0] max depth, [1] max parents
  // node checks (fold batches): op, arity and children, input
  const int *node_op, *node_input;
  int num_inputs;
};

// The walk, from the leaves on the list: emit(v, depth) once for every node that it reaches; finished and deepest are
// this thread's.  All links are in place (a barrier starts it).
template <class L, class EMIT>
__device__ __forceinline__ void walk_graph(const L& g, GraphShared& sh, const EMIT& emit, int& finished, int& deepest) {
  const int t = threadIdx.x, T = blockDim.x;
  finished = 0;
  deepest = 0;
  for (int lo = 0;;) {
    __syncthreads();
    const int hi = sh.tail;
    __syncthreads();
    if (lo == hi) break;
    for (int i = lo + t; i < hi; i += T) {
      int v = g.list[i], d = g.get_depth(v);
      unsigned h = g.get_head(v);
      while (true) {
        emit(v, d);
        ++finished;
        int nv = -1, nd = 0;
        unsigned nh = L::kNone;
        if (h & L::kSingle) {  // the parent's own link is read along with the report: one LDS latency a step
          const int p = (int)(h & ~L::kSingle);
          nh = g.get_head(p);
          if (g.arrive(p, d + 1, nd)) nv = p;
        } else if (h != L::kNone) {
          unsigned nx;
          int p = g.get_edge(h, nx);
          while (true) {  // the next edge is read along with the report
            const bool more = nx != L::kNone;
            unsigned nx2 = L::kNone;
            const int p2 = more ? g.get_edge(nx, nx2) : 0;
            int dp;
            if (g.arrive(p, d + 1, dp)) {
              int other = p, od = dp;
              if (nv < 0 || p < nv) other = nv, od = nd, nv = p, nd = dp;
              if (other >= 0) {
                g.set_depth(other, od);
                g.list[atomicAdd(&sh.tail, 1)] = other;
              }
            }
            if (!more) break;
            p = p2, nx = nx2;
          }
          if (nv >= 0) nh = g.get_head(nv);
        }
        if (nv < 0) break;
        v = nv, d = nd, h = nh;
      }
      deepest = max(deepest, d);  // a chain's last node is its deepest
    }
    lo = hi;
  }
}

// every thread's totals into sh
__device__ __forceinline__ void graph_totals(GraphShared& sh, int finished, int deepest, int parents) {
  for (int s = kWave / 2; s; s >>= 1) {
    finished += __shfl_xor(finished, s);
    deepest = max(deepest, __shfl_xor(deepest, s));
    parents = max(parents, __shfl_xor(parents, s));
  }
  if ((threadIdx.x & (kWave - 1)) == 0) {
    atomicAdd(&sh.done, finished);
    atomicMax(&sh.deepest, deepest);
    atomicMax(&sh.parents, parents);
  }
}

// Links the graph (nodes g0 .. g0 + n - 1, edges e0 .. e0 + e - 1) and, for a fold batch, checks every node first
// (the lowest node with an error counts, and its first check).
template <class L, bool CHECK>
__device__ __forceinline__ void run_graph(const L& g, const GraphArgs& a, const OpTable& ops, GraphShared& sh, int g0,
                                          int n, int e0, int e) {
  const int t = threadIdx.x, T = blockDim.x;
  for (int v = t; v < n; v += T) g.set_head(v, L::kNone);
  if (t == 0) sh = {0, 0, 0, 0, 0};
  __syncthreads();
  for (int v = t; v < n; v += T) {
    const int lo = a.cp[g0 + v], hi = a.cp[g0 + v + 1];
    if constexpr (CHECK) {
      int fault = 0;
      const int op = a.node_op[g0 + v], inp = a.node_input[g0 + v];
      if (op < 0 || op >= ops.n) {
        fault = FOLD_E_OP;
      } else if (hi - lo != ops.arity(op)) {
        fault = FOLD_E_ARITY;
      } else {
        for (int j = lo; j < hi; ++j)
          if (a.ci[j] != -1 && (a.ci[j] < g0 || a.ci[j] >= g0 + n)) fault = FOLD_E_CHILD;
        if (!fault && (ops.has_input(op) ? inp < 0 || inp >= a.num_inputs : inp != -1)) fault = FOLD_E_INPUT;
      }
      if (fault) {
        report(a.err, g0 + v + 1, fault);
        sh.bad = 1;
        continue;
      }
    }
    int children = 0;
    for (int j = lo; j < hi; ++j) {
      const int c = a.ci[j] - g0;
      if (a.ci[j] < 0) continue;
      ++children;
      g.set_edge(j - e0, v, g.link(c, j - e0));
    }
    if (children) {
      g.wait_for(v, children);
    } else {
      g.set_depth(v, 1);
      g.list[atomicAdd(&sh.tail, 1)] = v;
    }
  }
  __syncthreads();
  if (sh.bad) return;
  int parents = 0;
  for (int v = t; v < n; v += T) {
    const int k = close_node(g, v);
    a.indeg[g0 + v] = k;
    parents = max(parents, k);
  }
  int finished, deepest;
  walk_graph(g, sh, [&](int v, int d) { a.depth[g0 + v] = d; }, finished, deepest);
  graph_totals(sh, finished, deepest, parents);
  __syncthreads();
  if (t == 0) {
    if (sh.done < n) {
      report(a.cycle, g0 + 1, FOLD_E_CYCLE);
    } else {  // most graphs find the batch's maxima there already
      if (sh.deepest > __hip_atomic_load(&a.meta[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(&a.meta[0], sh.deepest);
      if (sh.parents > __hip_atomic_load(&a.meta[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(&a.meta[1], sh.parents);
    }
  }
}

// The pointer arrays have been checked.  CHECK (fold batches, at most two children): the nodes are checked here;
// without it their children have been checked too.  lds_bytes: dynamic LDS for the links.
template <bool CHECK, int THREADS>
__global__ __launch_bounds__(THREADS) void k_graph_depth(GraphArgs a, OpTable ops, int lds_bytes) {
  if (__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 8 == 0) return;  // a pointer array
  // Another graph's cycle does not end this one (the lowest cyclic graph counts), and must not: it can come in while this
  // workgroup starts, and then only the waves that read the word later would leave.  Errors of the checks are all in.
  if constexpr (!CHECK) {
    const unsigned long long e = __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (e != kNoErr && (e & 0xff) != (unsigned)-FOLD_E_CYCLE) return;
  }
  extern __shared__ __attribute__((aligned(16))) char links[];
  __shared__ GraphShared sh;
  const int g = blockIdx.x;
  const int g0 = a.gp[g], n = a.gp[g + 1] - g0;
  if (n == 0) return;
  const int e0 = a.cp[g0], e = a.cp[g0 + n] - e0;
  using LL = LdsLinks<CHECK>;
  using GL = GlobLinks<CHECK>;
  const bool fits = n < (int)LL::kNone && e < (int)LL::kNone && n * LL::kNodeBytes + e * LL::kEdgeBytes <= lds_bytes;
  if (fits)
    run_graph<LL, CHECK>(LL(links, n, e), a, ops, sh, g0, n, e0, e);
  else
    run_graph<GL, CHECK>(GL(a.scratch + GL::kNodeInts * (size_t)g0 + GL::kEdgeInts * (size_t)e0, n, e), a, ops, sh, g0,
                         n, e0, e);
}

template <bool CHECK>
void launch_graph_depth(const GraphArgs& a, const OpTable& ops, long long N, int G, int lds_bytes, hipStream_t st) {
  switch (graph_threads(N, G)) {
    case 128: hipLaunchKernelGGL((k_graph_depth<CHECK, 128>), dim3(G), dim3(128), lds_bytes, st, a, ops, lds_bytes); break;
    case 256: hipLaunchKernelGGL((k_graph_depth<CHECK, 256>), dim3(G), dim3(256), lds_bytes, st, a, ops, lds_bytes); break;
    default: hipLaunchKernelGGL((k_graph_depth<CHECK, 1024>), dim3(G), dim3(1024), lds_bytes, st, a, ops, lds_bytes); break;
  }
}

// LDS for the links of a graph: twice what an average graph takes, at least what a tree of 1,000 nodes takes (eleven
// such workgroups fit a compute unit) and at most 60 KB; larger graphs use scratch memory
inline int graph_lds_bytes(long long N, long long E, int G, int node_bytes, int edge_bytes) {
  const long long mean = (N * node_bytes + E * edge_bytes) / std::max(G, 1);
  return (int)std::min<long long>(61440, (std::max<long long>(1000 * (node_bytes + edge_bytes), 2 * mean) + 255) / 256 * 256);
}

// ---------------------------------------------------------------- device-wide exclusive scan

// blockIdx.y: one of several arrays of n, side by side (their partial sums and totals too)
__global__ void k_scan_reduce(const int* in, int n, int* partial) {
  const int b = blockIdx.x, t = threadIdx.x;
  in += (size_t)blockIdx.y * n;
  const long long base = (long long)b * kScanTile + (long long)t * kScanItems;
  int s = 0;
  for (int i = 0; i < kScanItems; ++i) {
    long long j = base + i;
    if (j < n) s += in[j];
  }
  s = block_sum<kBlock>(s);
  if (t == 0) partial[blockIdx.y * gridDim.x + b] = s;
}

// every workgroup adds up the sums of the tiles before its own (a launch less than a scan of them)
__global__ void k_scan_down(const int* in, int n, const int* partial, int* out, int* total) {
  const int b = blockIdx.x, t = threadIdx.x;
  in += (size_t)blockIdx.y * n;
  out += (size_t)blockIdx.y * n;
  partial += blockIdx.y * gridDim.x;
  const long long base = (long long)b * kScanTile + (long long)t * kScanItems;
  int v[kScanItems];
  int s = 0, before = 0;
  for (int i = t; i < b; i += kBlock) before += partial[i];
  for (int i = 0; i < kScanItems; ++i) {
    long long j = base + i;
    v[i] = j < n ? in[j] : 0;
    s += v[i];
  }
  before = block_sum<kBlock>(before);
  int tot;
  int pre = block_exscan<kBlock>(s, &tot) + before;
  for (int i = 0; i < kScanItems; ++i) {
    long long j = base + i;
    if (j < n) out[j] = pre;
    pre += v[i];
  }
  if (b == (int)gridDim.x - 1 && t == 0) total[blockIdx.y] = before + tot;
}

// exclusive scans of `rows` arrays of n, in -> out (may alias), their totals -> total[0 .. rows) (device); temp holds
// rows * ceil(n / tile) ints
void scan_exclusive(const int* in, int* out, int n, int rows, int* total, int* temp, hipStream_t st) {
  const int nb = std::max(1, (n + kScanTile - 1) / kScanTile);
  hipLaunchKernelGGL(k_scan_reduce, dim3(nb, rows), dim3(kBlock), 0, st, in, n, temp);
  hipLaunchKernelGGL(k_scan_down, dim3(nb, rows), dim3(kBlock), 0, st, in, n, temp, out, total);
}

// ---------------------------------------------------------------- stable LSD radix sort

// Work of a tile: kTileThreads threads, kTileItems items each; a wave owns consecutive items, 64 to a round.
__device__ __forceinline__ int tile_item(int r) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  return (w * kTileItems + r) * kWave + lane;
}
__device__ __forceinline__ unsigned long long lanes_below() { return (1ull << (threadIdx.x & (kWave - 1))) - 1; }

// Stable ranks: rank[r] = earlier items of this wave with the same digit d[r] (-1: no item); `mine` (this wave's
// counters, zero before) ends as the wave's count of every digit.  One ballot per digit bit finds a round's equal
// digits; rounds go in item order, so no barrier is needed inside a wave.
__device__ __forceinline__ void wave_ranks(volatile uint16_t* mine, const int (&d)[kTileItems], int bits,
                                           int (&rank)[kTileItems]) {
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    unsigned long long m = __ballot(d[r] >= 0);
    for (int b = 0; b < bits; ++b) {
      const int on = (d[r] >> b) & 1;
      const unsigned long long bal = __ballot(on);
      m &= on ? bal : ~bal;
    }
    const int below = __popcll(m & lanes_below());
    const int before = d[r] >= 0 ? mine[d[r]] : 0;
    __builtin_amdgcn_wave_barrier();
    if (d[r] >= 0 && below == 0) mine[d[r]] = (uint16_t)(before + __popcll(m));
    __builtin_amdgcn_wave_barrier();
    rank[r] = before + below;
  }
}

// the waves' counts of digit d become the counts of the waves before; returns the tile's count
__device__ __forceinline__ int scan_waves(uint16_t* counts, int stride, int d) {
  int run = 0;
  for (int w = 0; w < kTileThreads / kWave; ++w) {
    const int c = counts[w * stride + d];
    counts[w * stride + d] = (uint16_t)run;
    run += c;
  }
  return run;
}

// Whether a pass of a sort runs: never once the error word is set; with meta (the sort by depth and op) only if the
// depth found on the device, meta[0], gives keys with bits in the pass's digit.  The host launches as many passes as
// N * num_ops keys could need; sorted_buffer() says which buffer the last one that ran wrote.
struct SortGate {
  const unsigned long long* err;
  const int* meta;
  int num_ops, pass;
  __device__ __forceinline__ bool off() const {
    if (*err != kNoErr) return true;
    return meta && pass > 0 && (((long long)meta[0] * num_ops - 1) >> (kDigitBits * pass)) == 0;
  }
};
__device__ __forceinline__ int sorted_buffer(const int* meta, int num_ops) {
  const long long top = (long long)meta[0] * num_ops - 1;
  return (top >> kDigitBits) != 0 && (top >> (2 * kDigitBits)) == 0 ? 1 : 0;
}

// what a pass sorts: the nodes by depth and op, or the (key, value) pairs that an earlier pass left
struct NodeKeys {
  typedef unsigned Key;
  const int *depth, *op;
  int num_ops;
  __device__ __forceinline__ unsigned key(int i) const { return (unsigned)((depth[i] - 1) * num_ops + op[i]); }
  __device__ __forceinline__ int val(int i) const { return i; }
};
template <class K>
struct PairKeys {
  typedef K Key;
  const K* k;
  const int* v;
  __device__ __forceinline__ K key(int i) const { return k[i]; }
  __device__ __forceinline__ int val(int i) const { return v[i]; }
};

// n items (n_ptr: their number on the device, at most n)
struct SortSize {
  int n;
  const int* n_ptr;
  __device__ __forceinline__ int get() const { return n_ptr ? *n_ptr : n; }
};

// A cycle counts where no check failed; keys past kMaxKeys are an error.  Every workgroup of the sort's first launch
// finds that by itself, the later launches see the error word.
__device__ __forceinline__ bool sort_starts(unsigned long long* err, const unsigned long long* cycle, const int* meta,
                                            int num_ops) {
  if (*err != kNoErr) return false;
  if (*cycle != kNoErr) {
    if (threadIdx.x == 0) atomicMin(err, *cycle);
    return false;
  }
  if ((long long)meta[0] * num_ops > kMaxKeys) {
    if (threadIdx.x == 0) report(err, kTooDeep, FOLD_E_INVALID);
    return false;
  }
  return true;
}

// counts[b * kDigits + d] = items of tile b with digit d
template <class SRC, bool FIRST>
__global__ __launch_bounds__(kTileThreads) void k_sort_count(SRC src, SortSize size, int shift, int* counts, SortGate gate,
                                                             unsigned long long* err, const unsigned long long* cycle) {
  if (FIRST ? !sort_starts(err, cycle, gate.meta, gate.num_ops) : gate.off()) return;
  __shared__ int hist[kDigits];
  const int n = size.get(), b = blockIdx.x, t = threadIdx.x;
  if ((long long)b * kTile >= n) return;
  for (int d = t; d < kDigits; d += kTileThreads) hist[d] = 0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int i = b * kTile + r * kTileThreads + t;
    if (i < n) atomicAdd(&hist[(int)(src.key(i) >> shift) & (kDigits - 1)], 1);
  }
  __syncthreads();
  for (int d = t; d < kDigits; d += kTileThreads) counts[(size_t)b * kDigits + d] = hist[d];
}

// counts down every digit's column become the counts of the tiles before; the totals go to row B.  A workgroup takes
// 64 digits: 16 segments of tiles are summed, then rewritten.
__global__ __launch_bounds__(1024) void k_sort_columns(SortSize size, int* counts, int B, SortGate gate) {
  if (gate.off()) return;
  __shared__ int part[16][64];
  const int d = blockIdx.x * 64 + (threadIdx.x & 63), seg = threadIdx.x >> 6;
  const int nb = (size.get() + kTile - 1) / kTile, per = (nb + 15) / 16;
  const int lo = min(nb, seg * per), hi = min(nb, lo + per);
  int s = 0;
  for (int b = lo; b < hi; ++b) s += counts[(size_t)b * kDigits + d];
  part[seg][threadIdx.x & 63] = s;
  __syncthreads();
  int run = 0;
  for (int k = 0; k < seg; ++k) run += part[k][threadIdx.x & 63];
  for (int b = lo; b < hi; ++b) {
    const int c = counts[(size_t)b * kDigits + d];
    counts[(size_t)b * kDigits + d] = run;
    run += c;
  }
  if (seg == 15) counts[(size_t)B * kDigits + d] = run;
}

// Scatter of one pass.  B > kSelfTiles: the counts have been scanned down the columns.
template <class SRC>
__global__ __launch_bounds__(kTileThreads) void k_sort_scatter(SRC src, SortSize size, int shift, const int* counts, int B,
                                                               typename SRC::Key* keys_out, int* vals_out,
                                                               SortGate gate) {
  if (gate.off()) return;
  const int n = size.get(), b = blockIdx.x, t = threadIdx.x;
  if ((long long)b * kTile >= n) return;
  __shared__ uint16_t wcount[kTileThreads / kWave][kDigits];
  __shared__ int base[kDigits];
  typename SRC::Key key[kTileItems];
  int val[kTileItems], d[kTileItems], rank[kTileItems];
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int i = b * kTile + tile_item(r);
    const bool in = i < n;
    key[r] = in ? src.key(i) : 0;
    val[r] = in ? src.val(i) : 0;
    d[r] = in ? (int)(key[r] >> shift) & (kDigits - 1) : -1;
  }
  for (int i = t; i < (int)sizeof(wcount) / 4; i += kTileThreads) reinterpret_cast<uint32_t*>(&wcount[0][0])[i] = 0;
  static_assert(kDigits == 2 * kTileThreads, "two digits a thread");
  const int2* col = reinterpret_cast<const int2*>(counts) + t;
  int2 before = make_int2(0, 0), total = make_int2(0, 0);
  if (B > kSelfTiles) {
    before = col[(size_t)b * kTileThreads];
    total = col[(size_t)B * kTileThreads];
  } else {
    const int nb = (n + kTile - 1) / kTile;
#pragma unroll 8
    for (int k = 0; k < nb; ++k) {
      const int2 c = col[(size_t)k * kTileThreads];
      if (k < b) before.x += c.x, before.y += c.y;
      total.x += c.x, total.y += c.y;
    }
  }
  int all;
  const int first = block_exscan<kTileThreads>(total.x + total.y, &all);  // its barriers publish the zeroed counters
  base[2 * t] = first + before.x;
  base[2 * t + 1] = first + total.x + before.y;
  wave_ranks(wcount[t / kWave], d, kDigitBits, rank);
  __syncthreads();
  for (int k = t; k < kDigits; k += kTileThreads) (void)scan_waves(&wcount[0][0], kDigits, k);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    if (d[r] < 0) continue;
    const int at = base[d[r]] + wcount[t / kWave][d[r]] + rank[r];
    keys_out[at] = key[r];
    vals_out[at] = val[r];
  }
}

// one pass: count, column scan where there are many tiles, scatter; counts holds (B + 1) * kDigits ints
template <class SRC, bool FIRST = false>
void sort_pass(SRC src, SortSize size, int shift, int* counts, typename SRC::Key* keys_out, int* vals_out, SortGate gate,
               unsigned long long* err, const unsigned long long* cycle, hipStream_t st) {
  const int B = (size.n + kTile - 1) / kTile;
  hipLaunchKernelGGL((k_sort_count<SRC, FIRST>), dim3(B), dim3(kTileThreads), 0, st, src, size, shift, counts, gate, err,
                     cycle);
  if (B > kSelfTiles)
    hipLaunchKernelGGL(k_sort_columns, dim3(kDigits / 64), dim3(1024), 0, st, size, counts, B, gate);
  hipLaunchKernelGGL((k_sort_scatter<SRC>), dim3(B), dim3(kTileThreads), 0, st, src, size, shift, counts, B, keys_out,
                     vals_out, gate);
}
inline int sort_passes(unsigned long long max_key) {
  int passes = 1;
  while (max_key >> (kDigitBits * passes)) ++passes;
  return passes;
}

// ---------------------------------------------------------------- emission

// Everything after the sort, in two passes over the tiles of sorted nodes: the first writes what needs no prefix and
// sums per tile (group starts, edges, roots of the same range of node ids, rows of every op); in the second a tile
// adds up the sums of the tiles before it (a few KB from the L2) and writes every index.  Separate scans, gathers and
// sorts for these took about twenty launches.
struct EmitArgs {
  // the sort's two buffers
  const unsigned* keys[2];
  const int* vals[2];
  const int *cp, *ci, *node_input, *indeg;
  int N, num_ops, tiles;
  unsigned* link;                          // [N] by node: pool row, kOneParent where it has one parent edge
  int *starts, *edges, *roots, *op_count;  // [tiles] each; op_count [tiles][num_ops]
  int* moved;                              // [2][N] by group: the slot's children are not consecutive single rows
  int *pos_node, *node_pos, *gid, *level_ptr, *g_level, *g_op, *g_row_begin, *g_idx_off, *g_cbase0, *g_cbase1;
  int *child_pos, *child_one, *input_idx, *pos_npar, *root_pos, *op_rows, *op_cpos, *op_inp;
  unsigned long long* tok_key;  // rows that read the leaf table, by (op, row): (input op's number << 32) | leaf-table row
  int* tok_val;                 // ... and their pool rows
  int* meta;                    // [4] groups, [5] roots, [6] entries of tok_key
  const unsigned long long* err;
};

constexpr unsigned kOneParent = 0x80000000u;

// the op table in LDS: a lane's op indexes it, and from the kernel's arguments that is a load from memory
__device__ __forceinline__ void copy_ops(unsigned char* to, const OpTable& ops) {
  for (int o = threadIdx.x; o < ops.n; o += kTileThreads) to[o] = ops.bits[o];
}

__global__ __launch_bounds__(kTileThreads) void k_emit_sums(EmitArgs a, OpTable ops) {
  if (*a.err != kNoErr) return;
  __shared__ int rows[kMaxOps];
  __shared__ unsigned char bits[kMaxOps];
  copy_ops(bits, ops);
  const int b = blockIdx.x, t = threadIdx.x, buf = sorted_buffer(a.meta, a.num_ops);
  const unsigned* keys = a.keys[buf];
  for (int o = t; o < a.num_ops; o += kTileThreads) rows[o] = 0;
  __syncthreads();
  int starts = 0, edges = 0, roots = 0;
  const int p0 = b * kTile, p1 = min(a.N, p0 + kTile);
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int p = p0 + r * kTileThreads + t;
    if (p >= p1) continue;
    const int v = a.vals[buf][p];
    const unsigned key = keys[p], prev = p > 0 ? keys[p - 1] : ~0u, next = p + 1 < a.N ? keys[p + 1] : ~0u;
    const int level = (int)(key / (unsigned)a.num_ops), op = (int)(key - (unsigned)level * a.num_ops);
    const int parents = a.indeg[v];
    a.pos_node[p] = v;
    a.node_pos[v] = p;
    a.link[v] = (unsigned)p | (parents == 1 ? kOneParent : 0u);
    a.pos_npar[p] = parents;
    a.moved[p] = 0;
    a.moved[a.N + p] = 0;
    if (p == 0 || (int)(prev / (unsigned)a.num_ops) != level) a.level_ptr[level] = p;
    if (p == a.N - 1) a.level_ptr[level + 1] = a.N;
    starts += prev != key;  // ~0u is no key
    edges += bits[op] & 3;
    roots += a.indeg[p] == 0;
    // rows of an op: the ends of its runs in the tile minus their starts
    if (p == p0 || prev != key) atomicAdd(&rows[op], p0 - p);
    if (p == p1 - 1 || next != key) atomicAdd(&rows[op], p + 1 - p0);
  }
  starts = block_sum<kTileThreads>(starts);
  edges = block_sum<kTileThreads>(edges);
  roots = block_sum<kTileThreads>(roots);
  if (t == 0) {
    a.starts[b] = starts;
    a.edges[b] = edges;
    a.roots[b] = roots;
  }
  for (int o = t; o < a.num_ops; o += kTileThreads) a.op_count[(size_t)b * a.num_ops + o] = rows[o];
}

__global__ __launch_bounds__(kTileThreads) void k_emit(EmitArgs a, OpTable ops) {
  if (*a.err != kNoErr) return;
  constexpr int kWaves = kTileThreads / kWave;
  __shared__ uint16_t wcount[kWaves][kMaxOps];
  __shared__ int op_at[kMaxOps], op_total[kMaxOps], tok_at[kMaxOps], tok_op[kMaxOps];
  __shared__ int wsum[3][kWaves];
  __shared__ unsigned char bits[kMaxOps];
  copy_ops(bits, ops);
  const int b = blockIdx.x, t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
  const int buf = sorted_buffer(a.meta, a.num_ops);
  const unsigned* keys = a.keys[buf];
  const int* vals = a.vals[buf];
  for (int i = t; i < (int)sizeof(wcount) / 4; i += kTileThreads) reinterpret_cast<uint32_t*>(&wcount[0][0])[i] = 0;
  for (int o = t; o < kMaxOps; o += kTileThreads) op_at[o] = op_total[o] = 0;
  __syncthreads();
  // sums of the tiles before this one; rows of every op before it and in all
  int starts = 0, edges = 0, roots = 0;
  for (int k = t; k < b; k += kTileThreads) {
    starts += a.starts[k];
    edges += a.edges[k];
    roots += a.roots[k];
  }
  {
    int span = 1;
    while (span < a.num_ops) span <<= 1;
    const int o = t & (span - 1), parts = kTileThreads / span;
    int before = 0, total = 0;
    if (o < a.num_ops)
      for (int k = t / span; k < a.tiles; k += parts) {
        const int c = a.op_count[(size_t)k * a.num_ops + o];
        if (k < b) before += c;
        total += c;
      }
    for (int d = kWave / 2; d >= span; d >>= 1) {  // few ops: add up the wave's parts first
      before += __shfl_xor(before, d);
      total += __shfl_xor(total, d);
    }
    if (lane < span) {
      if (before) atomicAdd(&op_at[o], before);
      if (total) atomicAdd(&op_total[o], total);
    }
  }
  starts = block_sum<kTileThreads>(starts);
  edges = block_sum<kTileThreads>(edges);
  roots = block_sum<kTileThreads>(roots);
  {
    const bool is_op = t < a.num_ops, reads = is_op && (bits[t] & 4);
    const int before = is_op ? op_at[t] : 0, total = is_op ? op_total[t] : 0;
    int all, entries, n;
    const int first = block_exscan<kTileThreads>(total, &all);
    const int tok_first = block_exscan<kTileThreads>(reads ? total : 0, &entries);
    const int number = block_exscan<kTileThreads>(reads ? 1 : 0, &n);
    if (is_op) {
      op_at[t] = first + before;
      tok_at[t] = tok_first - first;  // entry of tok_key minus entry of op_rows
      tok_op[t] = reads ? number : -1;
    }
    if (b == 0 && t == 0) a.meta[6] = entries;
  }
  __syncthreads();
  // this tile's items
  int key_[kTileItems], node[kTileItems], op[kTileItems], rank[kTileItems];
  int s_at[kTileItems], e_at[kTileItems], r_at[kTileItems];
  bool start[kTileItems], root[kTileItems];
  int ws = 0, we = 0, wr = 0;
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int p = b * kTile + tile_item(r);
    const bool in = p < a.N;
    const unsigned key = in ? keys[p] : 0u;
    key_[r] = (int)key;
    node[r] = in ? vals[p] : -1;
    op[r] = in ? (int)(key % (unsigned)a.num_ops) : -1;
    start[r] = in && (p == 0 || keys[p - 1] != key);
    root[r] = in && a.indeg[p] == 0;
    const int arity = in ? bits[op[r]] & 3 : 0;
    const unsigned long long ms = __ballot(start[r]), m1 = __ballot(arity & 1), m2 = __ballot(arity & 2),
                             mr = __ballot(root[r]), lt = lanes_below();
    s_at[r] = ws + __popcll(ms & lt);
    e_at[r] = we + __popcll(m1 & lt) + 2 * __popcll(m2 & lt);
    r_at[r] = wr + __popcll(mr & lt);
    ws += __popcll(ms);
    we += __popcll(m1) + 2 * __popcll(m2);
    wr += __popcll(mr);
  }
  if (lane == 0) wsum[0][w] = ws, wsum[1][w] = we, wsum[2][w] = wr;
  int op_bits = 0;
  while ((1 << op_bits) < a.num_ops) ++op_bits;
  wave_ranks(wcount[w], op, op_bits, rank);
  __syncthreads();
  for (int o = t; o < a.num_ops; o += kTileThreads) (void)scan_waves(&wcount[0][0], kMaxOps, o);
  for (int k = 0; k < kWaves; ++k) {
    if (k < w) starts += wsum[0][k], edges += wsum[1][k], roots += wsum[2][k];
  }
  __syncthreads();
  if (b == a.tiles - 1 && t == kTileThreads - 1) {  // the last wave: everything before it, and its own
    a.meta[4] = starts + ws;
    a.meta[5] = roots + wr;
  }
  // every item's loads go out before any of its stores: chains of three (the node's edges, their nodes, those nodes'
  // rows), four items at once
  int c0[kTileItems], input[kTileItems], root_at[kTileItems];
  int c[kTileItems][2], cpos[kTileItems][2], one[kTileItems][2], prev0[2] = {-1, -1};
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int v = max(node[r], 0), p = b * kTile + tile_item(r);
    c0[r] = a.cp[v];
    input[r] = a.node_input[v];
    root_at[r] = root[r] ? a.node_pos[p] : 0;
  }
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int arity = node[r] >= 0 ? bits[op[r]] & 3 : 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) c[r][k] = k < arity ? a.ci[c0[r] + k] : -1;
  }
#pragma unroll
  for (int r = 0; r < kTileItems; ++r)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const unsigned x = c[r][k] >= 0 ? a.link[c[r][k]] : 0u;  // row and parent flag in one gather
      cpos[r][k] = c[r][k] >= 0 ? (int)(x & ~kOneParent) : -1;
      one[r][k] = (x & kOneParent) != 0;
    }
  // Static-graph layout of a child slot: its children are consecutive pool rows with one parent edge each (a batch
  // of identically shaped graphs with one operation per node position, i.e. manual batching, has it on every slot;
  // the kernels then address them as base + row).  The group's first row proposes its child as the base, a row
  // whose child does not follow the previous row's withdraws it.  (prev0: the child of the row before the wave's.)
  if (lane == 0 && node[0] >= 0 && !start[0]) {
    const int q0 = a.cp[vals[b * kTile + tile_item(0) - 1]];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int x = k < (bits[op[0]] & 3) ? a.ci[q0 + k] : -1;
      prev0[k] = x >= 0 ? a.node_pos[x] : -1;
    }
  }
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int p = b * kTile + tile_item(r);
    const bool in = node[r] >= 0;
    const int arity = in ? bits[op[r]] & 3 : 0;
    const int g = starts + s_at[r] + (start[r] ? 1 : 0) - 1, off = edges + e_at[r];
    int prev[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int up = __shfl_up(cpos[r][k], 1), last = __shfl(cpos[r > 0 ? r - 1 : 0][k], kWave - 1);
      prev[k] = lane > 0 ? up : (r > 0 ? last : prev0[k]);
    }
    if (!in) continue;
    a.gid[p] = g;
    if (start[r]) {
      a.g_level[g] = (int)((unsigned)key_[r] / (unsigned)a.num_ops) + 1;
      a.g_op[g] = op[r];
      a.g_row_begin[g] = p;
      a.g_idx_off[g] = off;
      a.g_cbase0[g] = one[r][0] ? cpos[r][0] : -1;
      a.g_cbase1[g] = one[r][1] ? cpos[r][1] : -1;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (k < arity) {
        a.child_pos[off + k] = cpos[r][k];
        a.child_one[off + k] = one[r][k];
        if (!start[r] && (!one[r][k] || cpos[r][k] != prev[k] + 1)) a.moved[(size_t)k * a.N + g] = 1;
      }
    const int q = op_at[op[r]] + wcount[w][op[r]] + rank[r];
    a.input_idx[p] = input[r];
    a.op_rows[q] = p;
    a.op_cpos[2 * (size_t)q] = cpos[r][0];
    a.op_cpos[2 * (size_t)q + 1] = cpos[r][1];
    a.op_inp[q] = input[r];
    if (tok_op[op[r]] >= 0) {
      a.tok_key[q + tok_at[op[r]]] = (unsigned long long)tok_op[op[r]] << 32 | (unsigned)input[r];
      a.tok_val[q + tok_at[op[r]]] = p;
    }
    if (root[r]) a.root_pos[roots + r_at[r]] = root_at[r];
  }
}

// The leaf-table gradient adds dz . W_in^T of every row into its leaf-table row; it is linear in dz, so the
// backward first sums dz over the rows of each (op, leaf-table row) and contracts once per distinct row.  The rows
// that read the leaf table are sorted by (op, leaf-table row), and the runs of equal keys are listed: starts per tile,
// then every entry's run.
__global__ __launch_bounds__(kTileThreads) void k_tok_sums(const unsigned long long* key, const int* n_ptr, int* starts,
                                                           const unsigned long long* err) {
  if (*err != kNoErr) return;
  const int n = *n_ptr, b = blockIdx.x;
  int s = 0;
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int i = b * kTile + r * kTileThreads + threadIdx.x;
    if (i < n) s += i == 0 || key[i - 1] != key[i];
  }
  s = block_sum<kTileThreads>(s);
  if (threadIdx.x == 0) starts[b] = s;
}

__global__ __launch_bounds__(kTileThreads) void k_tok_emit(const unsigned long long* key, const int* n_ptr,
                                                           const int* starts, int* tok_start, int* tok_row, int* tok_seg,
                                                           int* number_runs, const unsigned long long* err) {
  if (*err != kNoErr) return;
  const int n = *n_ptr, b = blockIdx.x, t = threadIdx.x;
  if ((long long)b * kTile >= n) return;
  __shared__ int wsum[kTileThreads / kWave], runs[kMaxOps];
  for (int o = t; o < kMaxOps; o += kTileThreads) runs[o] = 0;
  int before = 0;
  for (int k = t; k < b; k += kTileThreads) before += starts[k];
  before = block_sum<kTileThreads>(before);
  unsigned long long k_[kTileItems];
  int at[kTileItems], sum = 0;
  bool start[kTileItems];
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int i = b * kTile + tile_item(r);
    k_[r] = i < n ? key[i] : ~0ull;
    start[r] = i < n && (i == 0 || key[i - 1] != k_[r]);
    const unsigned long long m = __ballot(start[r]);
    at[r] = sum + __popcll(m & lanes_below());
    sum += __popcll(m);
  }
  if ((t & (kWave - 1)) == 0) wsum[t / kWave] = sum;
  __syncthreads();
  for (int k = 0; k < t / kWave; ++k) before += wsum[k];
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int i = b * kTile + tile_item(r);
    const int op = (int)(k_[r] >> 32);
    if (i < n) {
      const int u = before + at[r] + (start[r] ? 1 : 0) - 1;
      tok_seg[i] = u;
      if (start[r]) {
        tok_start[u] = i;
        tok_row[u] = (int)(unsigned)k_[r];
      }
      if (i == n - 1) tok_start[u + 1] = n;
    }
    // runs per input op: one add per op and round (the list is sorted by op), summed in LDS, then one add per op and
    // workgroup to the shared counter (an add per round from every wave: 54 us at 0.8 M entries, now 7)
    unsigned long long m = __ballot(start[r]);
    while (m) {
      const int leader = __ffsll((long long)m) - 1;
      const int lop = __shfl(op, leader);
      const unsigned long long same = __ballot(start[r] && op == lop);
      if ((t & (kWave - 1)) == leader) atomicAdd(&runs[lop], __popcll(same));
      m &= ~same;
    }
  }
  __syncthreads();
  for (int o = t; o < kMaxOps; o += kTileThreads)
    if (runs[o]) atomicAdd(&number_runs[o], runs[o]);
}

// error words "none", the meta words and `more` zero
__global__ void k_init_meta(void* em, int words, int* more, int n_more) {
  if (threadIdx.x < 2) static_cast<unsigned long long*>(em)[threadIdx.x] = kNoErr;
  int* meta = reinterpret_cast<int*>(static_cast<unsigned long long*>(em) + 2);
  for (int i = threadIdx.x; i < words; i += blockDim.x) meta[i] = 0;
  for (int i = threadIdx.x; i < n_more; i += blockDim.x) more[i] = 0;
}

// The one read-back of a schedule: the error word and meta, then the first lcap + 1 entries of level_ptr
// and the first gcap groups of each group array, side by side.
constexpr int kHdr = 16;
constexpr int kGroupArrays = 7;
struct GroupArrays {
  const int* a[kGroupArrays];  // level, op, row_begin, rows, idx_off, child base of slot 0, of slot 1
};
// (several workgroups: the group rows and child bases are finished here)
__global__ void k_finish(const unsigned long long* err, const int* meta, const int* level_ptr, GroupArrays garr, int N,
                         const int* moved, int* g_rows, int* cb0, int* cb1, int lcap, int gcap, const int* op_runs,
                         int num_ops, int* out) {
  const unsigned long long e = *err;
  const int i0 = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
  if (i0 == 0) {
    out[0] = (int)(unsigned)(e & 0xffffffffull);
    out[1] = (int)(unsigned)(e >> 32);
    for (int i = 0; i < 8; ++i) out[2 + i] = meta[i];
  }
  if (e != kNoErr) return;
  const int ng = N > 0 ? meta[4] : 0, nl = N > 0 ? min(meta[0] + 1, lcap + 1) : 0;
  for (int i = i0; i < nl; i += step) out[kHdr + i] = level_ptr[i];
  int* go = out + kHdr + lcap + 1;
  for (int g = i0; g < ng; g += step) {
    const int begin = garr.a[2][g], rows = (g + 1 < ng ? garr.a[2][g + 1] : N) - begin;
    const int c0 = moved[g] ? -1 : cb0[g], c1 = moved[N + g] ? -1 : cb1[g];
    g_rows[g] = rows;
    cb0[g] = c0;
    cb1[g] = c1;
    if (g >= gcap) continue;
    const int row[kGroupArrays] = {garr.a[0][g], garr.a[1][g], begin, rows, garr.a[4][g], c0, c1};
#pragma unroll
    for (int k = 0; k < kGroupArrays; ++k) go[k * gcap + g] = row[k];
  }
  for (int o = i0; o < num_ops; o += step) go[kGroupArrays * gcap + o] = op_runs[o];
}

// ---------------------------------------------------------------- a small batch in one launch
// A batch of up to 4,096 nodes is a chain of launches with almost no work in them (17, about 60 us), so one workgroup
// does all of it in LDS: the same steps as above, with barriers for launches (152 nodes in one kernel of 27 us, the
// schedule and the forward of eight levels 112 -> 90 us; 2,322 nodes in 45 us, with fourteen levels 222 -> 196).  It is
// bound by those barriers and the dependent LDS and memory accesses between them; past 4,096 nodes (or 8,192 edges or
// graphs) the arrays no longer fit and one compute unit is too few.
constexpr int kSmallThreads = 1024, kSmallWaves = kSmallThreads / kWave;
constexpr int kSmallNodes = 4096, kSmallEdges = 8192;

struct SmallArgs {
  const int *gp, *cp, *ci, *node_op, *node_input;
  int G, N, E, num_inputs;
  int *depth, *node_pos, *pos_node, *input_idx, *root_pos, *child_pos, *child_one, *gid, *pos_npar, *op_rows, *op_cpos,
      *op_inp, *tok_rows, *tok_seg, *tok_start, *tok_row, *level_ptr, *g_level, *g_op, *g_row_begin, *g_rows, *g_idx_off,
      *g_cbase0, *g_cbase1;
  int row_passes, tok_passes;  // digits of a leaf-table row; with one more where several ops read the table (0: none does)
  int lcap, gcap;
  int* out;
};

struct SmallLds {
  uint32_t head[kSmallNodes], state[kSmallNodes];  // links and depths; then ops by row, and the sorted keys
  uint32_t edge[kSmallEdges];                      // links; then the waves' digit counts
  uint16_t list[kSmallNodes];                      // links; then the groups' withdrawn child bases
  uint32_t keys[kSmallNodes];                      // each node's graph; then the sort's keys
  uint16_t vals[kSmallNodes], pos[kSmallNodes], parents[kSmallNodes], child[2][kSmallNodes], start[kSmallNodes],
      offset[kSmallNodes];
  int base[kDigits];
  int op_total[kMaxOps], op_at[kMaxOps], tok_at[kMaxOps], tok_op[kMaxOps], runs[kMaxOps];
  int sums[3][kSmallWaves];
  unsigned char bits[kMaxOps];
  unsigned long long err, cycle;
  GraphShared sh;
};
static_assert(sizeof(SmallLds) <= 160 * 1024, "the LDS of a compute unit");
static_assert(kSmallWaves * kDigits * 2 <= kSmallEdges * 4, "the digit counts take the edges' place");

// One stable pass over n (key, value) pairs in registers, item (wave, round, lane) in that order; through keys / vals.
template <class DIGIT>
__device__ __forceinline__ void small_pass(SmallLds& s, int n, int rounds, unsigned (&key)[kTileItems],
                                           int (&val)[kTileItems], const DIGIT& digit) {
  const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
  uint16_t* counts = reinterpret_cast<uint16_t*>(s.edge);
  for (int i = t; i < kSmallWaves * kDigits / 2; i += kSmallThreads) s.edge[i] = 0;
  int d[kTileItems], rank[kTileItems];
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int i = (w * rounds + r) * kWave + lane;
    d[r] = r < rounds && i < n ? digit(key[r], val[r]) : -1;
  }
  __syncthreads();
  wave_ranks(counts + w * kDigits, d, kDigitBits, rank);
  __syncthreads();
  int run = 0, all;
  for (int k = 0; k < kSmallWaves; ++k) {
    const int c = counts[k * kDigits + t];
    counts[k * kDigits + t] = (uint16_t)run;
    run += c;
  }
  s.base[t] = block_exscan<kSmallThreads>(run, &all);
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kTileItems; ++r)
    if (d[r] >= 0) {
      const int at = s.base[d[r]] + counts[w * kDigits + d[r]] + rank[r];
      s.keys[at] = key[r];
      s.vals[at] = (uint16_t)val[r];
    }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int i = (w * rounds + r) * kWave + lane;
    if (r < rounds && i < n) key[r] = s.keys[i], val[r] = s.vals[i];
  }
}

__global__ __launch_bounds__(kSmallThreads) void k_schedule_small(SmallArgs a, OpTable ops) {
  static_assert(kDigits == kSmallThreads, "one digit a thread");
  __shared__ SmallLds s;
  const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave, N = a.N, K = ops.n;
  const int rounds = (N + kSmallThreads - 1) / kSmallThreads;
  auto item = [&](int r) { return (w * rounds + r) * kWave + lane; };
  auto done = [&](unsigned long long e) {  // the error word alone
    if (t == 0) {
      a.out[0] = (int)(unsigned)(e & 0xffffffffull);
      a.out[1] = (int)(unsigned)(e >> 32);
    }
  };
  // pointers; keys[v] = the end of the graph that starts at node v (0: none does)
  if (t == 0) {
    s.err = s.cycle = kNoErr;
    s.sh = {0, 0, 0, 0, 0};
  }
  for (int o = t; o < kMaxOps; o += kSmallThreads) s.op_total[o] = s.runs[o] = 0;
  for (int o = t; o < K; o += kSmallThreads) s.bits[o] = ops.bits[o];
  for (int v = t; v < N; v += kSmallThreads) {
    s.head[v] = LdsLinks<true>::kNone;
    s.keys[v] = 0;
  }
  __syncthreads();
  bool bad = t == 0 && (a.gp[0] != 0 || a.gp[a.G] != N || a.cp[0] != 0 || a.cp[N] != a.E);
  for (int g = t; g < a.G; g += kSmallThreads) {
    const int lo = a.gp[g], hi = a.gp[g + 1];
    if (lo < 0 || hi > N || lo > hi) bad = true;
    else if (lo < hi) s.keys[lo] = (unsigned)hi;
  }
  for (int v = t; v < N; v += kSmallThreads) {
    const int lo = a.cp[v], hi = a.cp[v + 1];
    if (lo < 0 || hi > a.E || lo > hi) bad = true;
  }
  if (bad) s.sh.bad = 1;
  __syncthreads();
  if (s.sh.bad) {
    done((unsigned long long)(-FOLD_E_INVALID));
    return;
  }
  // the first node of every node's graph: the last graph start up to it
  int first[kTileItems], carry = 0;
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int v = item(r);
    int m = r < rounds && v < N && s.keys[v] ? v : 0;
    for (int d = 1; d < kWave; d <<= 1) {
      const int up = __shfl_up(m, d);
      if (lane >= d) m = max(m, up);
    }
    first[r] = max(m, carry);
    carry = max(carry, __shfl(m, kWave - 1));
  }
  if (lane == 0) s.sums[0][w] = carry;
  __syncthreads();
  for (int k = 0; k < w; ++k)
#pragma unroll
    for (int r = 0; r < kTileItems; ++r) first[r] = max(first[r], s.sums[0][k]);
  // node checks and links
  LdsLinks<true> g;
  g.state = s.state, g.head = s.head, g.edge = s.edge, g.depth = s.edge, g.list = s.list;
  int op_[kTileItems], c0[kTileItems], input[kTileItems];
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int v = item(r);
    const bool in = r < rounds && v < N;
    op_[r] = in ? a.node_op[v] : 0;
    input[r] = in ? a.node_input[v] : -1;
    c0[r] = in ? a.cp[v] : 0;
    if (!in) continue;
    const int lo = c0[r], hi = a.cp[v + 1], g0 = first[r], g1 = (int)s.keys[g0];
    int fault = 0;
    if (op_[r] < 0 || op_[r] >= K) {
      fault = FOLD_E_OP;
    } else if (hi - lo != (s.bits[op_[r]] & 3)) {
      fault = FOLD_E_ARITY;
    } else {
      for (int j = lo; j < hi; ++j)
        if (a.ci[j] != -1 && (a.ci[j] < g0 || a.ci[j] >= g1)) fault = FOLD_E_CHILD;
      if (!fault && (s.bits[op_[r]] & 4 ? input[r] < 0 || input[r] >= a.num_inputs : input[r] != -1))
        fault = FOLD_E_INPUT;
    }
    if (fault) {
      report(&s.err, v + 1, fault);
      continue;
    }
    int children = 0;
    for (int j = lo; j < hi; ++j)
      if (a.ci[j] >= 0) {
        ++children;
        g.set_edge(j, v, g.link(a.ci[j], j));
      }
    if (children) {
      g.wait_for(v, children);
    } else {
      g.set_depth(v, 1);
      g.list[atomicAdd(&s.sh.tail, 1)] = (uint16_t)v;
    }
  }
  __syncthreads();
  if (s.err != kNoErr) {
    done(s.err);
    return;
  }
  int most = 0;
  for (int v = t; v < N; v += kSmallThreads) {
    const int k = g.close(v);
    s.parents[v] = (uint16_t)k;
    most = max(most, k);
  }
  int finished, deepest;
  walk_graph(g, s.sh, [&](int v, int d) { g.set_depth(v, d); }, finished, deepest);
  graph_totals(s.sh, finished, deepest, most);
  __syncthreads();
  if (s.sh.done < N) {  // the lowest graph with a node that no walk finished (its state is no depth)
#pragma unroll
    for (int r = 0; r < kTileItems; ++r) {
      const int v = item(r);
      if (r < rounds && v < N && (s.state[v] == 0 || s.state[v] >> 24)) report(&s.cycle, first[r] + 1, FOLD_E_CYCLE);
    }
    __syncthreads();
    done(s.cycle);
    return;
  }
  const int D = s.sh.deepest;
  // sort by depth and op
  unsigned key[kTileItems];
  int val[kTileItems];
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int v = item(r);
    const bool in = r < rounds && v < N;
    const int d = in ? (int)s.state[v] : 1;
    key[r] = (unsigned)((d - 1) * K + op_[r]);
    val[r] = v;
    if (in) a.depth[v] = d;
  }
  __syncthreads();
  for (int shift = 0; shift == 0 || ((long long)D * K - 1) >> shift; shift += kDigitBits)
    small_pass(s, N, rounds, key, val, [&](unsigned k, int) { return (int)(k >> shift) & (kDigits - 1); });
  // rows, group starts, edges, roots
  unsigned char* row_op = reinterpret_cast<unsigned char*>(s.head);
  unsigned* moved = reinterpret_cast<unsigned*>(s.list);  // [2][kSmallNodes / 32] bits by group
  for (int i = t; i < kSmallNodes / 16; i += kSmallThreads) moved[i] = 0;
  int s_at[kTileItems], e_at[kTileItems], r_at[kTileItems], ws = 0, we = 0, wr = 0;
  bool start[kTileItems], root[kTileItems];
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int p = item(r);
    const bool in = r < rounds && p < N;
    const int level = (int)(key[r] / (unsigned)K);
    op_[r] = in ? (int)(key[r] - (unsigned)level * K) : -1;
    const unsigned prev = in && p > 0 ? s.keys[p - 1] : ~0u;
    start[r] = in && prev != key[r];
    root[r] = in && s.parents[p] == 0;
    const int arity = in ? s.bits[op_[r]] & 3 : 0;
    if (in) {
      s.state[p] = key[r];
      row_op[p] = (unsigned char)op_[r];
      s.pos[val[r]] = (uint16_t)p;
      a.pos_node[p] = val[r];
      a.node_pos[val[r]] = p;
      a.pos_npar[p] = s.parents[val[r]];
      if (p == 0 || (int)(prev / (unsigned)K) != level) {
        a.level_ptr[level] = p;
        if (level <= a.lcap) a.out[kHdr + level] = p;
      }
      if (p == N - 1) {
        a.level_ptr[level + 1] = N;
        if (level + 1 <= a.lcap) a.out[kHdr + level + 1] = N;
      }
      const unsigned next = p + 1 < N ? s.keys[p + 1] : ~0u;  // rows of an op: its runs' ends minus their starts
      if (start[r]) atomicAdd(&s.op_total[op_[r]], -p);
      if (next != key[r]) atomicAdd(&s.op_total[op_[r]], p + 1);
    }
    const unsigned long long ms = __ballot(start[r]), m1 = __ballot(arity & 1), m2 = __ballot(arity & 2),
                             mr = __ballot(root[r]), lt = lanes_below();
    s_at[r] = ws + __popcll(ms & lt);
    e_at[r] = we + __popcll(m1 & lt) + 2 * __popcll(m2 & lt);
    r_at[r] = wr + __popcll(mr & lt);
    ws += __popcll(ms);
    we += __popcll(m1) + 2 * __popcll(m2);
    wr += __popcll(mr);
  }
  if (lane == 0) s.sums[0][w] = ws, s.sums[1][w] = we, s.sums[2][w] = wr;
  // ranks within each op (the digit counts' place, cleared first)
  uint16_t* counts = reinterpret_cast<uint16_t*>(s.edge);
  for (int i = t; i < kSmallWaves * kMaxOps / 2; i += kSmallThreads) s.edge[i] = 0;
  __syncthreads();
  int rank[kTileItems], op_bits = 0;
  while ((1 << op_bits) < K) ++op_bits;
  wave_ranks(counts + w * kMaxOps, op_, op_bits, rank);
  {
    const bool is_op = t < K, reads = is_op && (s.bits[t] & 4);
    const int total = is_op ? s.op_total[t] : 0;
    int all, entries, n;
    const int at = block_exscan<kSmallThreads>(total, &all);
    const int tok = block_exscan<kSmallThreads>(reads ? total : 0, &entries);
    const int number = block_exscan<kSmallThreads>(reads ? 1 : 0, &n);
    if (is_op) {
      s.op_at[t] = at;
      s.tok_at[t] = tok - at;
      s.tok_op[t] = reads ? number : -1;
      int run = 0;
      for (int k = 0; k < kSmallWaves; ++k) {
        const int c = counts[k * kMaxOps + t];
        counts[k * kMaxOps + t] = (uint16_t)run;
        run += c;
      }
    }
    if (t == 0) s.base[0] = entries;
  }
  __syncthreads();
  const int entries = s.base[0];
  int starts = 0, edges = 0, roots = 0, num_groups = 0, num_roots = 0;
  for (int k = 0; k < kSmallWaves; ++k) {
    if (k < w) starts += s.sums[0][k], edges += s.sums[1][k], roots += s.sums[2][k];
    num_groups += s.sums[0][k];
    num_roots += s.sums[2][k];
  }
  // every index; child[k][p]: the child's row, 0x4000 where it has one parent edge, 0x8000 for no child
  constexpr unsigned kOne = 0x4000, kNoChild = 0x8000;
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int p = item(r);
    if (r >= rounds || p >= N) continue;
    const int v = val[r], arity = s.bits[op_[r]] & 3, gg = starts + s_at[r] + (start[r] ? 1 : 0) - 1, off = edges + e_at[r];
    const int at = a.cp[v], in_row = a.node_input[v], q = s.op_at[op_[r]] + counts[w * kMaxOps + op_[r]] + rank[r];
    int cpos[2] = {-1, -1};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int c = k < arity ? a.ci[at + k] : -1;
      const bool one = c >= 0 && s.parents[c] == 1;
      cpos[k] = c >= 0 ? (int)s.pos[c] : -1;
      s.child[k][p] = (uint16_t)(c >= 0 ? (unsigned)cpos[k] | (one ? kOne : 0u) : kNoChild);
      if (k < arity) {
        a.child_pos[off + k] = cpos[k];
        a.child_one[off + k] = one;
      }
    }
    if (start[r]) {
      s.start[gg] = (uint16_t)p;
      s.offset[gg] = (uint16_t)off;
    }
    c0[r] = gg;
    a.gid[p] = gg;
    a.input_idx[p] = in_row;
    a.op_rows[q] = p;
    a.op_cpos[2 * q] = cpos[0];
    a.op_cpos[2 * q + 1] = cpos[1];
    a.op_inp[q] = in_row;
    if (s.tok_op[op_[r]] >= 0) {  // in (op, row) order
      s.keys[q + s.tok_at[op_[r]]] = (unsigned)in_row;
      s.vals[q + s.tok_at[op_[r]]] = (uint16_t)p;
    }
    if (root[r]) a.root_pos[roots + r_at[r]] = s.pos[p];
  }
  __syncthreads();
  // child bases: withdrawn where a row's child does not follow the previous row's
#pragma unroll
  for (int r = 0; r < kTileItems; ++r) {
    const int p = item(r);
    if (r >= rounds || p >= N || start[r]) continue;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const unsigned x = s.child[k][p], before = s.child[k][p - 1];
      if (k < (s.bits[op_[r]] & 3) && (!(x & kOne) || (x & 0x3fff) != (before & 0x3fff) + 1))
        atomicOr(&moved[k * (kSmallNodes / 32) + (c0[r] >> 5)], 1u << (c0[r] & 31));
    }
  }
  __syncthreads();
  int* go = a.out + kHdr + a.lcap + 1;
  for (int gg = t; gg < num_groups; gg += kSmallThreads) {
    const int p = s.start[gg], rows = (gg + 1 < num_groups ? (int)s.start[gg + 1] : N) - p;
    const int level = (int)(s.state[p] / (unsigned)K) + 1, op = row_op[p];
    int cb[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const unsigned x = s.child[k][p];
      const bool ok = (x & kOne) && !(moved[k * (kSmallNodes / 32) + (gg >> 5)] >> (gg & 31) & 1);
      cb[k] = ok ? (int)(x & 0x3fff) : -1;
    }
    a.g_level[gg] = level;
    a.g_op[gg] = op;
    a.g_row_begin[gg] = p;
    a.g_rows[gg] = rows;
    a.g_idx_off[gg] = s.offset[gg];
    a.g_cbase0[gg] = cb[0];
    a.g_cbase1[gg] = cb[1];
    if (gg < a.gcap) {
      const int row[kGroupArrays] = {level, op, p, rows, (int)s.offset[gg], cb[0], cb[1]};
#pragma unroll
      for (int k = 0; k < kGroupArrays; ++k) go[k * a.gcap + gg] = row[k];
    }
  }
  // the rows that read the leaf table by (op, leaf-table row), and their runs
  if (a.tok_passes > 0) {
    const int n = entries, per = (n + kSmallThreads - 1) / kSmallThreads;
    auto entry = [&](int r) { return (w * per + r) * kWave + lane; };
#pragma unroll
    for (int r = 0; r < kTileItems; ++r) {
      const int i = entry(r);
      key[r] = r < per && i < n ? s.keys[i] : 0u;
      val[r] = r < per && i < n ? (int)s.vals[i] : 0;
    }
    __syncthreads();
    for (int ps = 0; ps < a.tok_passes; ++ps) {
      if (ps < a.row_passes)
        small_pass(s, n, per, key, val, [&](unsigned k, int) { return (int)(k >> (kDigitBits * ps)) & (kDigits - 1); });
      else
        small_pass(s, n, per, key, val, [&](unsigned, int p) { return s.tok_op[row_op[p]]; });
    }
    ws = 0;
#pragma unroll
    for (int r = 0; r < kTileItems; ++r) {
      const int i = entry(r);
      const bool in = r < per && i < n;
      start[r] = in && (i == 0 || s.keys[i - 1] != key[r] || row_op[s.vals[i - 1]] != row_op[val[r]]);
      const unsigned long long m = __ballot(start[r]);
      s_at[r] = ws + __popcll(m & lanes_below());
      ws += __popcll(m);
    }
    if (lane == 0) s.sums[0][w] = ws;
    __syncthreads();
    starts = 0;
    for (int k = 0; k < w; ++k) starts += s.sums[0][k];
#pragma unroll
    for (int r = 0; r < kTileItems; ++r) {
      const int i = entry(r);
      if (r >= per || i >= n) continue;
      const int u = starts + s_at[r] + (start[r] ? 1 : 0) - 1;
      a.tok_rows[i] = val[r];
      a.tok_seg[i] = u;
      if (start[r]) {
        a.tok_start[u] = i;
        a.tok_row[u] = (int)key[r];
        atomicAdd(&s.runs[s.tok_op[row_op[val[r]]]], 1);
      }
      if (i == n - 1) a.tok_start[u + 1] = n;
    }
  }
  __syncthreads();
  for (int o = t; o < K; o += kSmallThreads) go[kGroupArrays * a.gcap + o] = s.runs[o];
  if (t == 0) {
    done(kNoErr);
    int* meta = a.out + 2;
    meta[0] = D;
    meta[1] = s.sh.parents;
    meta[4] = num_groups;
    meta[5] = num_roots;
    meta[6] = entries;
  }
}

inline dim3 grid_for(long long n) { return dim3((unsigned)std::max(1LL, (n + kBlock - 1) / kBlock)); }

// Temporaries of one phase on one stream: the sizes are declared first (reserve), then one pooled block backs them all
// (commit).  The block and the read-back buffer go back to the pool at scope exit, once the stream has finished with
// them: finished() says that the call has waited already.
struct Temp {
  hipStream_t st;
  int device;
  void* block = nullptr;
  int* stage = nullptr;  // pinned, kStageInts ints
  bool waited = false;
  std::vector<std::pair<void**, size_t>> want;
  size_t bytes = 0;
  Temp(hipStream_t s, int dev) : st(s), device(dev) {}
  Temp(const Temp&) = delete;
  Temp& operator=(const Temp&) = delete;
  ~Temp() {
    if (!block && !stage) return;
    if (!waited && hipStreamSynchronize(st) != hipSuccess) return;  // a device in error: nothing is reused
    pool_free(device, block, false);
    stage_free(stage);
  }
  template <class T>
  void reserve(T** p, size_t count) {
    want.push_back({reinterpret_cast<void**>(p), bytes});
    bytes += (std::max<size_t>(count, 1) * sizeof(T) + 255) / 256 * 256;
  }
  bool commit(bool with_stage) {
    block = pool_alloc(device, std::max<size_t>(bytes, 256), false);
    if (with_stage) stage = stage_alloc();
    if (!block || (with_stage && !stage)) return false;
    for (auto& w : want) *w.first = static_cast<char*>(block) + w.second;
    return true;
  }
};

int decode_error(unsigned long long w, std::string* msg) {
  const int code = -(int)(w & 0xffull);
  const long long node = (long long)(w >> 8) - 1;
  if ((long long)(w >> 8) == kTooDeep) {
    *msg = "fold_schedule: depth * num_ops exceeds 2^30 (the sort keys)";
    return code;
  }
  const char* what = "invalid batch";
  switch (code) {
    case FOLD_E_INVALID: what = "graph_ptr / child_ptr malformed"; break;
    case FOLD_E_OP: what = "node_op out of range"; break;
    case FOLD_E_ARITY: what = "child count differs from the operation's arity"; break;
    case FOLD_E_CHILD: what = "child out of range or in another graph"; break;
    case FOLD_E_INPUT: what = "node_input inconsistent with has_input or out of range"; break;
    case FOLD_E_CYCLE: what = "graph contains a cycle"; break;
    default: break;
  }
  *msg = std::string("fold_schedule: ") + what + (node >= 0 ? " (node " + std::to_string(node) + ")" : "");
  return code;
}

}  // namespace

void sched_destroy_impl(fold_sched* h);
static void sched_destroy(fold_sched* h) { sched_destroy_impl(h); }

int32_t schedule_impl(const fold_batch* b, hipStream_t st, fold_sched** out) {
  const int N = b->num_nodes, E = b->num_edges, G = b->num_graphs, K = b->num_ops;
  for (int i = 0; i < K; ++i)
    if (b->ops[i].arity > 2) {
      set_error("fold_schedule: operations take at most two children");
      return FOLD_E_INVALID;
    }
  if (K > kMaxOps) {
    set_error("fold_schedule: at most 256 operations are supported");
    return FOLD_E_INVALID;
  }
  OpTable ops{};
  ops.n = K;
  for (int i = 0; i < K; ++i) {
    ops.bits[i] = (unsigned char)(b->ops[i].arity | (b->ops[i].has_input ? 4 : 0));
  }
  int device = 0;
  FOLD_HIP_CHECK(hipGetDevice(&device));

  auto* h = new fold_sched();
  Sched& s = h->s;
  s.N = N; s.E = E; s.G = G; s.num_ops = K; s.device = device; s.num_inputs = b->num_inputs;
  s.ops.assign(b->ops, b->ops + K);
  auto fail = [&](int code) {
    sched_destroy(h);
    return code;
  };

  // persistent arrays sized by N and E; the level and group tables take N + 1 and 5 x N entries (there are
  // at most N levels and N groups), so nothing waits for the depth to be known on the host
  const size_t n1 = (size_t)N * 23 + 2 * (size_t)E + 17;
  s.blob = pool_alloc(device, n1 * sizeof(int), true);
  if (!s.blob) {
    set_error("fold_schedule: out of device memory");
    return fail(FOLD_E_NOMEM);
  }
  const size_t cap = std::max<size_t>(N, 1);
  int* q = static_cast<int*>(s.blob);
  s.depth = q; q += N;
  s.node_pos = q; q += N;
  s.pos_node = q; q += N;
  s.input_idx = q; q += N;
  s.root_pos = q; q += N;
  s.child_pos = q; q += E;
  s.child_one = q; q += E;
  s.pos_group = q; q += N;
  s.pos_npar = q; q += N;
  s.op_rows = q; q += N;
  s.op_cpos = q; q += 2 * (size_t)N;
  s.op_inp = q; q += N;
  s.tok_rows = q; q += N;
  s.tok_seg = q; q += N;
  s.tok_start = q; q += N + 1;
  s.tok_row = q; q += N;
  s.level_ptr = q; q += cap + 1;
  s.g_level = q; q += cap;
  s.g_op = q; q += cap;
  s.g_row_begin = q; q += cap;
  s.g_rows = q; q += cap;
  s.g_idx_off = q; q += cap;
  s.g_cbase0 = q; q += cap;
  s.g_cbase1 = q; q += cap;

  // temporaries of the whole schedule, one pooled allocation
  Temp tmp(st, device);
  // err, then meta: [0] max depth, [1] max parents, [4] groups, [5] roots, [6] rows that read the leaf table
  struct ErrMeta {
    unsigned long long err, cycle;  // a cycle counts only where no node check failed
    int meta[8];
  };
  ErrMeta* em = nullptr;
  int *indeg = nullptr, *scratch = nullptr, *moved = nullptr;
  unsigned* link = nullptr;
  unsigned* keys[2] = {nullptr, nullptr};
  unsigned long long* tok_keys[2] = {nullptr, nullptr};
  int *vals[2] = {nullptr, nullptr}, *tok_vals[2] = {nullptr, nullptr};
  int *sort_counts = nullptr, *tile_sums = nullptr, *op_count = nullptr;
  const long long scratch_ints = GlobLinks<true>::kNodeInts * (long long)N + GlobLinks<true>::kEdgeInts * (long long)E;
  const int B = (N + kTile - 1) / kTile;
  int input_ops = 0;
  for (int i = 0; i < K; ++i) input_ops += b->ops[i].has_input ? 1 : 0;
  const bool any_input = input_ops > 0;
  constexpr int kLcap = 4096, kGcap = 4096;  // levels and groups read back with the error word
  static_assert(kHdr + (kLcap + 1) + kGroupArrays * (size_t)kGcap + kMaxOps <= kStageInts, "the read-back buffer");
  int* op_runs = nullptr;  // [kMaxOps] runs of equal (op, leaf-table row) of the ops that read the leaf table
  const bool small = N > 0 && N <= kSmallNodes && E <= kSmallEdges && G <= kSmallEdges;
  tmp.reserve(&em, 1);
  tmp.reserve(&op_runs, kMaxOps);
  if (N > 0 && !small) {
    tmp.reserve(&indeg, N);
    tmp.reserve(&scratch, (size_t)scratch_ints);
    tmp.reserve(&moved, 2 * (size_t)N);
    tmp.reserve(&link, N);
    for (int i = 0; i < 2; ++i) {
      tmp.reserve(&keys[i], N);
      tmp.reserve(&vals[i], N);
      if (any_input) {
        tmp.reserve(&tok_keys[i], N);
        tmp.reserve(&tok_vals[i], N);
      }
    }
    tmp.reserve(&sort_counts, (size_t)(B + 1) * kDigits);
    tmp.reserve(&tile_sums, 4 * (size_t)B);
    tmp.reserve(&op_count, (size_t)B * K);
  }
  if (!tmp.commit(true)) {
    set_error("fold_schedule: out of device memory (temporaries)");
    return fail(FOLD_E_NOMEM);
  }
  unsigned long long* err = &em->err;
  int* meta = em->meta;
  // digits of a leaf-table row, and one pass more over the op where several ops read the table
  const int row_passes = any_input ? sort_passes((unsigned long long)std::max(b->num_inputs - 1, 0)) : 0;
  const int tok_passes = row_passes + (input_ops > 1 ? 1 : 0);
  if (small) {
    SmallArgs a{};
    a.gp = b->graph_ptr; a.cp = b->child_ptr; a.ci = b->child_idx; a.node_op = b->node_op; a.node_input = b->node_input;
    a.G = G; a.N = N; a.E = E; a.num_inputs = b->num_inputs;
    a.depth = s.depth; a.node_pos = s.node_pos; a.pos_node = s.pos_node; a.input_idx = s.input_idx;
    a.root_pos = s.root_pos; a.child_pos = s.child_pos; a.child_one = s.child_one; a.gid = s.pos_group;
    a.pos_npar = s.pos_npar; a.op_rows = s.op_rows; a.op_cpos = s.op_cpos; a.op_inp = s.op_inp;
    a.tok_rows = s.tok_rows; a.tok_seg = s.tok_seg; a.tok_start = s.tok_start; a.tok_row = s.tok_row;
    a.level_ptr = s.level_ptr; a.g_level = s.g_level; a.g_op = s.g_op; a.g_row_begin = s.g_row_begin;
    a.g_rows = s.g_rows; a.g_idx_off = s.g_idx_off; a.g_cbase0 = s.g_cbase0; a.g_cbase1 = s.g_cbase1;
    a.row_passes = row_passes; a.tok_passes = tok_passes;
    a.lcap = kLcap; a.gcap = kGcap; a.out = tmp.stage;
    hipLaunchKernelGGL(k_schedule_small, dim3(1), dim3(kSmallThreads), 0, st, a, ops);
  } else {
    hipLaunchKernelGGL(k_init_meta, dim3(1), dim3(kBlock), 0, st, em, 8, op_runs, kMaxOps);
    hipLaunchKernelGGL(k_check_struct, grid_for(std::max(G + 1, N + 1)), dim3(kBlock), 0, st, b->graph_ptr, G,
                       b->child_ptr, N, E, err);
    if (N > 0) {
      if (G > 0) {
        const int lds = graph_lds_bytes(N, E, G, LdsLinks<true>::kNodeBytes, LdsLinks<true>::kEdgeBytes);
        const GraphArgs ga{b->graph_ptr, b->child_ptr, b->child_idx, s.depth, indeg, scratch, err, &em->cycle, meta,
                           b->node_op, b->node_input, b->num_inputs};
        launch_graph_depth<true>(ga, ops, N, G, lds, st);
      }

      // sort by (depth - 1) * num_ops + op: as many passes as N * num_ops keys could need are launched; those the actual
      // depth does not need return at once
      const unsigned long long max_key = std::min<unsigned long long>((unsigned long long)N * K,
                                                                      (unsigned long long)kMaxKeys) - 1;
      const int passes = sort_passes(max_key);
      const SortSize all{N, nullptr};
      for (int ps = 0; ps < passes; ++ps) {
        const SortGate gate{err, meta, K, ps};
        if (ps == 0)
          sort_pass<NodeKeys, true>({s.depth, b->node_op, K}, all, 0, sort_counts, keys[0], vals[0], gate, err, &em->cycle,
                                    st);
        else
          sort_pass<PairKeys<unsigned>>({keys[(ps - 1) & 1], vals[(ps - 1) & 1]}, all, kDigitBits * ps, sort_counts,
                                        keys[ps & 1], vals[ps & 1], gate, err, &em->cycle, st);
      }
      EmitArgs ea{};
      for (int i = 0; i < 2; ++i) {
        ea.keys[i] = keys[i];
        ea.vals[i] = vals[i];
      }
      ea.cp = b->child_ptr; ea.ci = b->child_idx; ea.node_input = b->node_input; ea.indeg = indeg;
      ea.N = N; ea.num_ops = K; ea.tiles = B;
      ea.starts = tile_sums; ea.edges = tile_sums + B; ea.roots = tile_sums + 2 * (size_t)B;
      ea.op_count = op_count; ea.moved = moved; ea.link = link;
      ea.pos_node = s.pos_node; ea.node_pos = s.node_pos; ea.gid = s.pos_group; ea.level_ptr = s.level_ptr;
      ea.g_level = s.g_level; ea.g_op = s.g_op; ea.g_row_begin = s.g_row_begin; ea.g_idx_off = s.g_idx_off;
      ea.g_cbase0 = s.g_cbase0; ea.g_cbase1 = s.g_cbase1;
      ea.child_pos = s.child_pos; ea.child_one = s.child_one; ea.input_idx = s.input_idx; ea.pos_npar = s.pos_npar;
      ea.root_pos = s.root_pos; ea.op_rows = s.op_rows; ea.op_cpos = s.op_cpos; ea.op_inp = s.op_inp;
      ea.tok_key = tok_keys[0]; ea.tok_val = tok_vals[0];
      ea.meta = meta; ea.err = err;
      hipLaunchKernelGGL(k_emit_sums, dim3(B), dim3(kTileThreads), 0, st, ea, ops);
      hipLaunchKernelGGL(k_emit, dim3(B), dim3(kTileThreads), 0, st, ea, ops);

      // the rows that read the leaf table in (op, leaf-table row) order, and their runs: they come in (op, row) order,
      // so passes over the leaf-table row's bits and, where several ops read it, one over the op sort them
      if (any_input) {
        const SortSize entries{N, meta + 6};
        for (int ps = 0; ps < tok_passes; ++ps) {
          const SortGate gate{err, nullptr, 0, 0};
          sort_pass<PairKeys<unsigned long long>>({tok_keys[ps & 1], tok_vals[ps & 1]}, entries,
                                                  ps < row_passes ? kDigitBits * ps : 32, sort_counts,
                                                  tok_keys[(ps + 1) & 1],
                                                  ps + 1 < tok_passes ? tok_vals[(ps + 1) & 1] : s.tok_rows, gate, err,
                                                  &em->cycle, st);
        }
        const unsigned long long* sorted = tok_keys[tok_passes & 1];
        int* tok_starts = tile_sums + 3 * (size_t)B;
        hipLaunchKernelGGL(k_tok_sums, dim3(B), dim3(kTileThreads), 0, st, sorted, meta + 6, tok_starts, err);
        hipLaunchKernelGGL(k_tok_emit, dim3(B), dim3(kTileThreads), 0, st, sorted, meta + 6, tok_starts, s.tok_start,
                           s.tok_row, s.tok_seg, op_runs, err);
      }
    }
  }
  GroupArrays ga{{s.g_level, s.g_op, s.g_row_begin, s.g_rows, s.g_idx_off, s.g_cbase0, s.g_cbase1}};
  // a workgroup per 1,024 possible groups, at most 16 (a batch has few groups; a thousand-level chain of them still
  // takes a few steps)
  if (!small)
    hipLaunchKernelGGL(k_finish, dim3(std::min(16, N / 1024 + 1)), dim3(kBlock), 0, st, err, meta, s.level_ptr, ga, N, moved,
                     s.g_rows, s.g_cbase0, s.g_cbase1, kLcap, kGcap, op_runs, K, tmp.stage);
  if (hipGetLastError() != hipSuccess) {
    set_error("fold_schedule: kernel launch failed");
    return fail(FOLD_E_DEVICE);
  }
  // the one synchronisation: error word, meta, and the level / group tables up to kLcap / kGcap entries
  if (hipStreamSynchronize(st) != hipSuccess) {
    set_error("fold_schedule: device error while scheduling");
    return fail(FOLD_E_DEVICE);
  }
  tmp.waited = true;
  const int* hb = tmp.stage;
  const unsigned long long ew = (unsigned long long)(unsigned)hb[0] | ((unsigned long long)(unsigned)hb[1] << 32);
  if (ew != kNoErr) {
    std::string msg;
    int code = decode_error(ew, &msg);
    set_error(msg);
    return fail(code);
  }
  const int* hm = hb + 2;
  const int D = N > 0 ? hm[0] : 0;
  const int ng = N > 0 ? hm[4] : 0;
  s.D = D;
  s.max_parents = N > 0 ? hm[1] : 0;
  s.num_groups = ng;
  s.R = N > 0 ? hm[5] : 0;
  if (N == 0) {
    s.h_level_ptr.assign(1, 0);
  } else if (D + 1 <= kLcap + 1 && ng <= kGcap) {
    const int* hl = hb + kHdr;
    s.h_level_ptr.assign(hl, hl + D + 1);
    const int* hg = hl + kLcap + 1;
    s.h_level.assign(hg, hg + ng);
    s.h_op.assign(hg + kGcap, hg + kGcap + ng);
    s.h_row_begin.assign(hg + 2 * kGcap, hg + 2 * kGcap + ng);
    s.h_rows.assign(hg + 3 * kGcap, hg + 3 * kGcap + ng);
    s.h_idx_off.assign(hg + 4 * kGcap, hg + 4 * kGcap + ng);
    s.h_cbase0.assign(hg + 5 * kGcap, hg + 5 * kGcap + ng);
    s.h_cbase1.assign(hg + 6 * kGcap, hg + 6 * kGcap + ng);
  } else {
    // more levels or groups than the first read-back holds: read the whole tables (a second synchronisation)
    s.h_level_ptr.resize(D + 1);
    std::vector<int>* dst[kGroupArrays] = {&s.h_level, &s.h_op, &s.h_row_begin, &s.h_rows, &s.h_idx_off,
                                           &s.h_cbase0, &s.h_cbase1};
    bool ok = hipMemcpyAsync(s.h_level_ptr.data(), s.level_ptr, (size_t)(D + 1) * sizeof(int),
                             hipMemcpyDeviceToHost, st) == hipSuccess;
    for (int k = 0; k < kGroupArrays; ++k) {
      dst[k]->resize(ng);
      ok = ok && hipMemcpyAsync(dst[k]->data(), ga.a[k], (size_t)ng * sizeof(int), hipMemcpyDeviceToHost, st) ==
                     hipSuccess;
    }
    if (!ok || hipStreamSynchronize(st) != hipSuccess) {
      set_error("fold_schedule: device error while reading the group table");
      return fail(FOLD_E_DEVICE);
    }
  }
  // ranges of op_rows per op, and of tok_rows and their runs per op that reads the leaf table
  s.h_op_row_ptr.assign(K + 1, 0);
  for (int g = 0; g < ng; ++g) s.h_op_row_ptr[s.h_op[g] + 1] += s.h_rows[g];
  s.h_tok_row_ptr.assign(K + 1, 0);
  s.h_tok_ptr.assign(K + 1, 0);
  const int* runs = hb + kHdr + (kLcap + 1) + kGroupArrays * kGcap;
  for (int o = 0; o < K; ++o) {
    const bool reads = N > 0 && b->ops[o].has_input;
    s.h_tok_row_ptr[o + 1] = s.h_tok_row_ptr[o] + (reads ? s.h_op_row_ptr[o + 1] : 0);
    s.h_tok_ptr[o + 1] = s.h_tok_ptr[o] + (reads ? *runs++ : 0);
  }
  for (int o = 0; o < K; ++o) s.h_op_row_ptr[o + 1] += s.h_op_row_ptr[o];
  *out = h;
  return FOLD_OK;
}

void sched_destroy_impl(fold_sched* h) {
  if (!h) return;
  if (h->s.blob) pool_free_after_wait(h->s.device, h->s.blob);
  delete h;
}

// ================================================================ the paper's form: typed states
// Section 2's five steps on a typed DAG (constants of a tensor type as sources, operations with typed inputs
// and outputs, edges from a specific output), with the pass-throughs and per-(depth, type) concatenations
// made explicit.  Phase 1 validates, takes depths (the per-graph depth kernel above, whose constants sit at
// 1: the paper's depth is one less), lists the values (node, output slot), finds each value's deepest
// reader and counts its pass-through instances; one read-back sizes phase 2.  Phase 2 emits the
// pass-through instances, sorts operation nodes and pass-throughs by (depth, operation) (stable: node ids,
// then value order), cuts the batches, lays out each depth's concatenation per type (operation order, then
// output slot, then batch order) and writes every gather index.

namespace {

constexpr int kMaxTypedOps = 64, kMaxTypes = 16, kMaxSlots = 8;

struct TypedOpTable {
  int K, T;
  unsigned char nin[kMaxTypedOps], nout[kMaxTypedOps];
  unsigned char in_type[kMaxTypedOps][kMaxSlots], out_type[kMaxTypedOps][kMaxSlots];
  unsigned char out_rank[kMaxTypedOps][kMaxSlots];  // rank of output k among the op's outputs of its type
  unsigned char nout_t[kMaxTypedOps][kMaxTypes];    // the op's outputs of type t
};

__device__ __forceinline__ int t_nout(const TypedOpTable& o, int op) { return op < 0 ? 1 : o.nout[op]; }

__global__ void k_typed_check(const int* node_op, const int* in_ptr, const int* in_node, const int* in_slot,
                              const int* node_graph, int N, TypedOpTable ops, unsigned long long* err) {
  // a pointer array; another node's error does not end this node's check (the lowest counts)
  if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 8 == 0) return;
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= N) return;
  const int op = node_op[v], a = in_ptr[v], b = in_ptr[v + 1];
  if (op < 0) {
    if (-1 - op >= ops.T) report(err, v + 1, FOLD_E_OP);
    else if (b != a) report(err, v + 1, FOLD_E_INVALID);
    return;
  }
  if (op >= ops.K) { report(err, v + 1, FOLD_E_OP); return; }
  if (b - a != ops.nin[op]) { report(err, v + 1, FOLD_E_INVALID); return; }
  for (int j = 0; j < b - a; ++j) {
    const int u = in_node[a + j], k = in_slot[a + j];
    if (u < 0 || u >= N) { report(err, v + 1, FOLD_E_INVALID); return; }
    if (node_graph[u] != node_graph[v]) { report(err, v + 1, FOLD_E_CHILD); return; }
    const int uop = node_op[u];
    if (uop >= ops.K || (uop < 0 && -1 - uop >= ops.T)) continue;  // that node reports its own error
    if (k < 0 || k >= t_nout(ops, uop)) { report(err, v + 1, FOLD_E_INVALID); return; }
    const int tu = uop < 0 ? -1 - uop : ops.out_type[uop][k];
    if (tu != ops.in_type[op][j]) { report(err, v + 1, FOLD_E_INVALID); return; }
  }
}

// paper depth (constants 0), the number of values of each node and of constants of each type; last[8 v + k] = the
// deepest depth that reads value k of node v (its own depth if nobody does)
__global__ void k_typed_nodes(const int* kdepth, const int* node_op, int N, TypedOpTable ops, int* depth,
                              int* nout_v, int* last, int* meta, const unsigned long long* err) {
  if (*err != kNoErr) return;
  // constants are counted in LDS first: an add per constant to one counter takes 370 us for 32,000 of them
  __shared__ int consts[kMaxTypes];
  if (threadIdx.x < kMaxTypes) consts[threadIdx.x] = 0;
  __syncthreads();
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v < N) {
    const int op = node_op[v], d = kdepth[v] - 1, n = t_nout(ops, op);
    depth[v] = d;
    nout_v[v] = n;
    for (int k = 0; k < n; ++k) last[(size_t)kMaxSlots * v + k] = d;
    if (op < 0) atomicAdd(&consts[-1 - op], 1);
  }
  __syncthreads();
  if (threadIdx.x < kMaxTypes && consts[threadIdx.x]) atomicAdd(&meta[8 + threadIdx.x], consts[threadIdx.x]);
}

__global__ void k_typed_last(const int* depth, const int* in_ptr, const int* in_node, const int* in_slot, int N,
                             int* last, const unsigned long long* err) {
  if (*err != kNoErr) return;
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= N) return;
  for (int e = in_ptr[v]; e < in_ptr[v + 1]; ++e)
    atomicMax(&last[(size_t)kMaxSlots * in_node[e] + in_slot[e]], depth[v]);
}

// pass-through instances of every node's values: one per depth strictly between a value's own and its deepest reader's
__device__ __forceinline__ int t_passes(const int* last, int v, int k, int d) {
  return max(0, last[(size_t)kMaxSlots * v + k] - d - 1);
}
__global__ void k_typed_npass(const int* depth, const int* nout_v, const int* last, int N, int* npass,
                              const unsigned long long* err) {
  if (*err != kNoErr) return;
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= N) return;
  int n = 0;
  for (int k = 0; k < nout_v[v]; ++k) n += t_passes(last, v, k, depth[v]);
  npass[v] = n;
}

// all of them in 64 bits (total starts at -1, the error word "none")
__global__ void k_typed_pass_total(const int* npass, int N, unsigned long long* total) {
  unsigned long long s = 0;
  for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < N; v += gridDim.x * blockDim.x) s += (unsigned)npass[v];
  for (int d = kWave / 2; d; d >>= 1) s += __shfl_xor(s, d);
  if ((threadIdx.x & (kWave - 1)) == 0 && s) atomicAdd(total, s);
}

// the instances, and the first one of every value
__global__ void k_typed_pass_emit(const int* depth, const int* nout_v, const int* val_ptr, const int* last,
                                  const int* node_pass, int N, int* pass_ptr, int* pass_node, int* pass_slot,
                                  int* pass_depth) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= N) return;
  int p = node_pass[v];
  for (int k = 0; k < nout_v[v]; ++k) {
    pass_ptr[val_ptr[v] + k] = p;
    const int n = t_passes(last, v, k, depth[v]);
    for (int j = 0; j < n; ++j, ++p) {
      pass_node[p] = v;
      pass_slot[p] = k;
      pass_depth[p] = depth[v] + 1 + j;
    }
  }
}

// sort keys (depth - 1) * (K + T) + op of operation nodes and pass-throughs (op K + t); constants of type t get
// `sent` + t, past every real key, and sort to the end by type
__global__ void k_typed_keys(const int* depth, const int* node_op, int N, const int* pass_node, const int* pass_slot,
                             const int* pass_depth, int P, TypedOpTable ops, unsigned sent, unsigned* keys,
                             int* vals) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int KT = ops.K + ops.T;
  if (i < N) {
    const int op = node_op[i];
    keys[i] = op < 0 ? sent + (unsigned)(-1 - op) : (unsigned)((depth[i] - 1) * KT + op);
    vals[i] = i;
  } else if (i < N + P) {
    const int p = i - N, u = pass_node[p], uop = node_op[u];
    const int t = uop < 0 ? -1 - uop : ops.out_type[uop][pass_slot[p]];
    keys[i] = (unsigned)((pass_depth[p] - 1) * KT + ops.K + t);
    vals[i] = i;
  }
}

// the items in order, then the constants: a constant's index in its concatenation is its rank in its type
__global__ void k_typed_items(const unsigned* keys, const int* vals, int M, int n, int N, unsigned sent,
                              const int* meta, const int* val_ptr, int* item_node, int* flag, int* vidx) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int x = vals[i];
  if (i >= M) {
    int rank = i - M;
    for (int t = 0; t < (int)(keys[i] - sent); ++t) rank -= meta[8 + t];
    vidx[val_ptr[x]] = rank;
    return;
  }
  item_node[i] = x < N ? x : -1 - (x - N);
  flag[i] = (i == 0 || keys[i] != keys[i - 1]) ? 1 : 0;
}

__global__ void k_typed_batches(const unsigned* keys, const int* flag, const int* exs, int M, int KT, int* bidx,
                                int* b_begin, int* b_depth, int* b_op) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M) return;
  const int b = exs[i] + flag[i] - 1;
  bidx[i] = b;
  if (flag[i]) {
    b_begin[b] = i;
    b_depth[b] = (int)(keys[i] / (unsigned)KT) + 1;
    b_op[b] = (int)(keys[i] % (unsigned)KT);
  }
}

// per batch (entries past the batch count get zeros): rows, per type t its outputs of type t (rows * the op's outputs
// of type t) at cnt[t * M + b], and its gather entries at cnt[T * M + b]
__global__ void k_typed_batch_sizes(const int* nb_ptr, int M, const int* b_begin, const int* b_op, TypedOpTable ops,
                                    int* b_rows, int* cnt) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= M) return;
  const int nb = *nb_ptr;
  if (b >= nb) {
    for (int t = 0; t <= ops.T; ++t) cnt[(size_t)t * M + b] = 0;
    return;
  }
  const int rows = (b + 1 < nb ? b_begin[b + 1] : M) - b_begin[b];
  const int op = b_op[b];
  b_rows[b] = rows;
  cnt[(size_t)ops.T * M + b] = rows * (op < ops.K ? ops.nin[op] : 1);
  for (int t = 0; t < ops.T; ++t)
    cnt[(size_t)t * M + b] = rows * (op < ops.K ? ops.nout_t[op][t] : (op - ops.K == t ? 1 : 0));
}

// first and last batch of every depth; the batches' gather offsets
__global__ void k_typed_depth_span(const int* nb_ptr, const int* b_depth, const int* goff, int* dfirst, int* dlast,
                                   int* b_goff) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  const int nb = *nb_ptr;
  if (b >= nb) return;
  const int d = b_depth[b];
  b_goff[b] = goff[b];
  if (b == 0 || b_depth[b - 1] != d) dfirst[d] = b;
  if (b == nb - 1 || b_depth[b + 1] != d) dlast[d] = b;
}

// state sizes: depth 0 from the constants per type (meta[8 + t]), deeper ones from the batch scans
__global__ void k_typed_state_size(int D, int M, int T, const int* dfirst, const int* dlast, const int* cnt,
                                   const int* cscan, const int* meta, int* size) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (D + 1) * T) return;
  const int d = i / T, t = i - d * T;
  if (d == 0) {
    size[i] = meta[8 + t];
    return;
  }
  const size_t o = (size_t)t * M;
  size[i] = cscan[o + dlast[d]] + cnt[o + dlast[d]] - cscan[o + dfirst[d]];
}

// concatenation index of every item's outputs at the item's depth: vidx[value] for operation nodes,
// pidx[p] for pass-through instance p
__global__ void k_typed_out_idx(const int* item_node, const int* bidx, const int* b_begin, const int* b_depth,
                                const int* b_op, const int* b_rows, const int* dfirst, const int* cscan, int M,
                                const int* val_ptr, TypedOpTable ops, int* vidx, int* pidx) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M) return;
  const int b = bidx[i], r = i - b_begin[b], op = b_op[b], rows = b_rows[b], f = dfirst[b_depth[b]];
  const int x = item_node[i];
  if (op < ops.K) {
    for (int k = 0; k < ops.nout[op]; ++k) {
      const size_t o = (size_t)ops.out_type[op][k] * M;
      vidx[val_ptr[x] + k] = cscan[o + b] - cscan[o + f] + ops.out_rank[op][k] * rows + r;
    }
  } else {
    const size_t o = (size_t)(op - ops.K) * M;
    pidx[-1 - x] = cscan[o + b] - cscan[o + f] + r;
  }
}

// the label index of value (u, k) read at depth d: the value itself if it was made at d - 1, else its
// pass-through instance at d - 1
__device__ __forceinline__ int typed_label(const int* depth, const int* val_ptr, const int* vidx, const int* pass_ptr,
                                           const int* pidx, int u, int k, int d) {
  const int du = depth[u], q = val_ptr[u] + k;
  return du == d - 1 ? vidx[q] : pidx[pass_ptr[q] + (d - 2 - du)];
}

__global__ void k_typed_gather(const int* item_node, const int* bidx, const int* b_begin, const int* b_depth,
                               const int* b_op, const int* b_rows, const int* b_goff, int M, const int* depth,
                               const int* in_ptr, const int* in_node, const int* in_slot, const int* val_ptr,
                               const int* vidx, const int* pass_ptr, const int* pidx, const int* pass_node,
                               const int* pass_slot, TypedOpTable ops, int* gather, int* edge_index) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M) return;
  const int b = bidx[i], r = i - b_begin[b], d = b_depth[b], rows = b_rows[b];
  const int x = item_node[i];
  int* g = gather + b_goff[b] + r;
  if (b_op[b] < ops.K) {
    for (int e = in_ptr[x], j = 0; e < in_ptr[x + 1]; ++e, ++j) {
      const int lab = typed_label(depth, val_ptr, vidx, pass_ptr, pidx, in_node[e], in_slot[e], d);
      g[j * rows] = lab;
      edge_index[e] = lab;
    }
  } else {
    const int p = -1 - x;
    g[0] = typed_label(depth, val_ptr, vidx, pass_ptr, pidx, pass_node[p], pass_slot[p], d);
  }
}

__global__ void k_typed_finish(const unsigned long long* err, const int* meta, const int* b_depth, const int* b_op,
                               const int* b_rows, const int* b_goff, const int* size, int M, int nsize, int cap,
                               int* out) {
  const unsigned long long e = *err;
  const int i0 = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
  if (i0 == 0) {
    out[0] = (int)(unsigned)(e & 0xffffffffull);
    out[1] = (int)(unsigned)(e >> 32);
    for (int i = 0; i < 14; ++i) out[2 + i] = meta[i];
  }
  if (e != kNoErr) return;
  const int n = M > 0 ? min(meta[4], cap) : 0, ns = min(nsize, cap);
  for (int i = i0; i < n; i += step) {
    out[kHdr + i] = b_depth[i];
    out[kHdr + cap + i] = b_op[i];
    out[kHdr + 2 * cap + i] = b_rows[i];
    out[kHdr + 3 * cap + i] = b_goff[i];
  }
  for (int i = i0; i < ns; i += step) out[kHdr + 4 * cap + i] = size[i];
}

}  // namespace

void typed_sched_destroy_impl(fold_typed_sched* h) {
  if (!h) return;
  if (h->t.blob) pool_free_after_wait(h->t.device, h->t.blob);
  delete h;
}

int32_t schedule_typed_impl(const fold_typed_batch* b, hipStream_t st, fold_typed_sched** out) {
  const int N = b->num_nodes, E = b->num_edges, G = b->num_graphs, K = b->num_ops, T = b->num_types;
  if (K < 1 || K > kMaxTypedOps || T < 1 || T > kMaxTypes) {
    set_error("fold_schedule_typed: need 1..64 operations and 1..16 types");
    return FOLD_E_INVALID;
  }
  TypedOpTable ops{};
  ops.K = K;
  ops.T = T;
  for (int o = 0; o < K; ++o) {
    const fold_typed_op& op = b->ops[o];
    if (op.num_inputs < 1 || op.num_inputs > kMaxSlots || op.num_outputs < 1 || op.num_outputs > kMaxSlots ||
        !op.in_type || !op.out_type) {
      set_error("fold_schedule_typed: operation " + std::to_string(o) + " needs 1..8 inputs and 1..8 outputs");
      return FOLD_E_INVALID;
    }
    ops.nin[o] = (unsigned char)op.num_inputs;
    ops.nout[o] = (unsigned char)op.num_outputs;
    for (int j = 0; j < op.num_inputs; ++j) {
      if (op.in_type[j] < 0 || op.in_type[j] >= T) {
        set_error("fold_schedule_typed: operation " + std::to_string(o) + " has an input type out of range");
        return FOLD_E_INVALID;
      }
      ops.in_type[o][j] = (unsigned char)op.in_type[j];
    }
    for (int k = 0; k < op.num_outputs; ++k) {
      const int t = op.out_type[k];
      if (t < 0 || t >= T) {
        set_error("fold_schedule_typed: operation " + std::to_string(o) + " has an output type out of range");
        return FOLD_E_INVALID;
      }
      ops.out_type[o][k] = (unsigned char)t;
      ops.out_rank[o][k] = ops.nout_t[o][t]++;
    }
  }
  int device = 0;
  FOLD_HIP_CHECK(hipGetDevice(&device));
  auto* h = new fold_typed_sched();
  TypedSched& s = h->t;
  s.N = N; s.E = E; s.K = K; s.T = T; s.device = device;
  auto fail = [&](int code) {
    typed_sched_destroy_impl(h);
    return code;
  };
  auto device_error = [&](const char* what) {
    set_error(std::string("fold_schedule_typed: ") + what);
    return fail(FOLD_E_DEVICE);
  };

  // phase 1 temporaries (kept to the end)
  Temp tmp1(st, device);
  struct ErrMeta {
    unsigned long long err, cycle;
    int meta[8 + kMaxTypes];  // [0] max depth + 1, [1] max parents, [2] values, [3] pass-throughs,
                              // [4] batches, [8 + t] constants of type t
  };
  static_assert(offsetof(ErrMeta, meta) == 2 * sizeof(unsigned long long), "k_init_meta's layout");
  ErrMeta* em = nullptr;
  int *node_graph = nullptr, *indeg = nullptr, *scratch = nullptr, *kdepth = nullptr, *depth = nullptr,
      *counts = nullptr, *offsets = nullptr, *last = nullptr, *scan_tmp1 = nullptr;  // values and pass-throughs by node
  tmp1.reserve(&em, 1);
  tmp1.reserve(&node_graph, N);
  tmp1.reserve(&indeg, N);
  tmp1.reserve(&scratch, GlobLinks<false>::kNodeInts * (size_t)N + GlobLinks<false>::kEdgeInts * (size_t)E);
  tmp1.reserve(&kdepth, N);
  tmp1.reserve(&depth, N);
  tmp1.reserve(&counts, 2 * (size_t)N);
  tmp1.reserve(&offsets, 2 * (size_t)N);
  tmp1.reserve(&last, kMaxSlots * (size_t)N);
  tmp1.reserve(&scan_tmp1, 2 * ((size_t)N / kScanTile + 2));
  if (!tmp1.commit(false)) {
    set_error("fold_schedule_typed: out of device memory (temporaries)");
    return fail(FOLD_E_NOMEM);
  }
  unsigned long long* err = &em->err;
  int* meta = em->meta;
  hipLaunchKernelGGL(k_init_meta, dim3(1), dim3(64), 0, st, em, 8 + kMaxTypes, nullptr, 0);
  int *nout_v = counts, *npass = counts + N, *val_ptr = offsets, *node_pass = offsets + N;
  hipLaunchKernelGGL(k_check_struct, grid_for(std::max(G + 1, N + 1)), dim3(kBlock), 0, st, b->graph_ptr, G,
                     b->in_ptr, N, E, err);
  if (N > 0) {
    if (G > 0) hipLaunchKernelGGL(k_node_graph, dim3(G), dim3(kBlock), 0, st, b->graph_ptr, node_graph, err);
    hipLaunchKernelGGL(k_typed_check, grid_for(N), dim3(kBlock), 0, st, b->node_op, b->in_ptr, b->in_node,
                       b->in_slot, node_graph, N, ops, err);
    if (G > 0) {
      const int lds = graph_lds_bytes(N, E, G, LdsLinks<false>::kNodeBytes, LdsLinks<false>::kEdgeBytes);
      const GraphArgs ga{b->graph_ptr, b->in_ptr, b->in_node, kdepth, indeg, scratch, err, err, meta, nullptr, nullptr,
                         0};
      launch_graph_depth<false>(ga, OpTable{}, N, G, lds, st);
    }
    hipLaunchKernelGGL(k_typed_nodes, grid_for(N), dim3(kBlock), 0, st, kdepth, b->node_op, N, ops, depth, nout_v,
                       last, meta, err);
    hipLaunchKernelGGL(k_typed_last, grid_for(N), dim3(kBlock), 0, st, depth, b->in_ptr, b->in_node, b->in_slot, N,
                       last, err);
    hipLaunchKernelGGL(k_typed_npass, grid_for(N), dim3(kBlock), 0, st, depth, nout_v, last, N, npass, err);
    scan_exclusive(counts, offsets, N, 2, meta + 2, scan_tmp1, st);
  }
  if (hipGetLastError() != hipSuccess) return device_error("kernel launch failed");
  // first synchronisation: the error word, the depth, and the sizes of phase 2 (no values where the error word is set)
  ErrMeta hm{};
  if (hipMemcpyAsync(&hm, em, sizeof(hm), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return device_error("device error while validating");
  if (hm.err != kNoErr) {
    std::string msg;
    int code = decode_error(hm.err, &msg);
    set_error("fold_schedule_typed" + msg.substr(msg.find(':')));
    return fail(code);
  }
  const int D = N > 0 ? hm.meta[0] - 1 : 0;
  const int V = N > 0 ? hm.meta[2] : 0;
  const int P = N > 0 ? hm.meta[3] : 0;
  // 32-bit counts hold the rows of any batch whose values could not pass through every depth; of the others (deep graphs)
  // the pass-throughs are counted again
  if ((long long)V * D + N + E > INT_MAX) {
    unsigned long long total = 0;
    hipLaunchKernelGGL(k_typed_pass_total, dim3(std::min(256, N / kBlock + 1)), dim3(kBlock), 0, st, npass, N, &em->cycle);
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(&total, &em->cycle, sizeof(total), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
      return device_error("device error while counting pass-throughs");
    if ((total += 1) + N + E > INT_MAX) {
      set_error("fold_schedule_typed: " + std::to_string(total) + " pass-throughs (rows and edges with them have to stay below 2^31)");
      return fail(FOLD_E_INVALID);
    }
  }
  if ((long long)(D + 1) * (K + T) > kMaxKeys) {
    set_error("fold_schedule_typed: depth * (operations + types) exceeds 2^30 (the sort keys)");
    return fail(FOLD_E_INVALID);
  }
  int nconst = 0;
  for (int t = 0; t < T; ++t) nconst += hm.meta[8 + t];
  const int M = N - nconst + P;  // items: operation nodes and pass-through instances
  s.D = D; s.P = P; s.M = M;
  const int ngather = E + P;
  s.ngather = ngather;

  // persistent arrays, now that P is known
  const size_t nsize = (size_t)(D + 1) * T;
  const size_t Mc = std::max(M, 1);
  const size_t n_int = (size_t)N + 6 * Mc + (size_t)std::max(ngather, 1) + 3 * (size_t)std::max(P, 1) + nsize +
                       (size_t)std::max(E, 1) + 16;
  s.blob = pool_alloc(device, n_int * sizeof(int), true);
  if (!s.blob) {
    set_error("fold_schedule_typed: out of device memory");
    return fail(FOLD_E_NOMEM);
  }
  int* q = static_cast<int*>(s.blob);
  s.depth = q; q += N;
  s.batch_depth = q; q += Mc;
  s.batch_op = q; q += Mc;
  s.batch_rows = q; q += Mc;
  s.batch_goff = q; q += Mc;
  s.batch_begin = q; q += Mc;
  s.item_node = q; q += Mc;
  s.gather = q; q += std::max(ngather, 1);
  s.pass_node = q; q += std::max(P, 1);
  s.pass_slot = q; q += std::max(P, 1);
  s.pass_depth = q; q += std::max(P, 1);
  s.state_size = q; q += nsize;
  s.edge_index = q; q += std::max(E, 1);
  if (N > 0 && hipMemcpyAsync(s.depth, depth, (size_t)N * sizeof(int), hipMemcpyDeviceToDevice, st) != hipSuccess)
    return device_error("copy of the depths failed");

  // phase 2
  const int NI = N + P;  // sort entries: every node (constants sort last) and every pass-through
  const int B = (NI + kTile - 1) / kTile;
  Temp tmp2(st, device);
  unsigned *ka = nullptr, *kb = nullptr;
  int *va = nullptr, *vb = nullptr, *flag = nullptr, *exs = nullptr, *sort_counts = nullptr, *scan_tmp = nullptr;
  int *bidx = nullptr, *pass_ptr = nullptr, *cnt = nullptr, *cscan = nullptr, *dspan = nullptr, *vidx = nullptr,
      *pidx = nullptr;
  constexpr int kCap = 4096;  // batches and state sizes read back with the final error word
  static_assert(kHdr + 5 * (size_t)kCap <= kStageInts, "the read-back buffer");
  tmp2.reserve(&ka, std::max(NI, 1));
  tmp2.reserve(&kb, std::max(NI, 1));
  tmp2.reserve(&va, std::max(NI, 1));
  tmp2.reserve(&vb, std::max(NI, 1));
  tmp2.reserve(&flag, std::max(NI, 1));
  tmp2.reserve(&exs, std::max(NI, 1));
  tmp2.reserve(&sort_counts, (size_t)(B + 1) * kDigits);
  tmp2.reserve(&scan_tmp, (size_t)(T + 1) * (Mc / kScanTile + 2));
  tmp2.reserve(&bidx, Mc);
  tmp2.reserve(&pass_ptr, std::max(V, 1));
  tmp2.reserve(&cnt, (size_t)(T + 1) * Mc);
  tmp2.reserve(&cscan, (size_t)(T + 1) * Mc);
  tmp2.reserve(&dspan, 2 * (size_t)(D + 1));
  tmp2.reserve(&vidx, std::max(V, 1));
  tmp2.reserve(&pidx, std::max(P, 1));
  int* totals = nullptr;  // of the scans, unused
  tmp2.reserve(&totals, T + 1);
  if (!tmp2.commit(true)) {
    set_error("fold_schedule_typed: out of device memory (temporaries)");
    return fail(FOLD_E_NOMEM);
  }
  int* dfirst = dspan;
  int* dlast = dspan + (D + 1);
  const int KT = K + T;
  if (N > 0) {
    if (P > 0)
      hipLaunchKernelGGL(k_typed_pass_emit, grid_for(N), dim3(kBlock), 0, st, depth, nout_v, val_ptr, last, node_pass, N,
                         pass_ptr, s.pass_node, s.pass_slot, s.pass_depth);
    const unsigned sent = (unsigned)(D * KT);
    hipLaunchKernelGGL(k_typed_keys, grid_for(NI), dim3(kBlock), 0, st, depth, b->node_op, N, s.pass_node,
                       s.pass_slot, s.pass_depth, P, ops, sent, ka, va);
    const int passes = sort_passes(sent + T - 1);
    for (int ps = 0; ps < passes; ++ps) {
      sort_pass<PairKeys<unsigned>>({ka, va}, {NI, nullptr}, kDigitBits * ps, sort_counts, kb, vb, {err, nullptr, 0, 0},
                                    err, &em->cycle, st);
      std::swap(ka, kb);
      std::swap(va, vb);
    }
    hipLaunchKernelGGL(k_typed_items, grid_for(NI), dim3(kBlock), 0, st, ka, va, M, NI, N, sent, meta, val_ptr,
                       s.item_node, flag, vidx);
    if (M > 0) {
      scan_exclusive(flag, exs, M, 1, meta + 4, scan_tmp, st);
      hipLaunchKernelGGL(k_typed_batches, grid_for(M), dim3(kBlock), 0, st, ka, flag, exs, M, KT, bidx,
                         s.batch_begin, s.batch_depth, s.batch_op);
      hipLaunchKernelGGL(k_typed_batch_sizes, grid_for(M), dim3(kBlock), 0, st, meta + 4, M, s.batch_begin,
                         s.batch_op, ops, s.batch_rows, cnt);
      scan_exclusive(cnt, cscan, M, T + 1, totals, scan_tmp, st);
      hipLaunchKernelGGL(k_typed_depth_span, grid_for(M), dim3(kBlock), 0, st, meta + 4, s.batch_depth,
                         cscan + (size_t)T * M, dfirst, dlast, s.batch_goff);
    }
    hipLaunchKernelGGL(k_typed_state_size, grid_for((long long)nsize), dim3(kBlock), 0, st, D, std::max(M, 1), T,
                       dfirst, dlast, cnt, cscan, meta, s.state_size);
    if (M > 0) {
      hipLaunchKernelGGL(k_typed_out_idx, grid_for(M), dim3(kBlock), 0, st, s.item_node, bidx, s.batch_begin,
                         s.batch_depth, s.batch_op, s.batch_rows, dfirst, cscan, M, val_ptr, ops, vidx, pidx);
      hipLaunchKernelGGL(k_typed_gather, grid_for(M), dim3(kBlock), 0, st, s.item_node, bidx, s.batch_begin,
                         s.batch_depth, s.batch_op, s.batch_rows, s.batch_goff, M, depth, b->in_ptr, b->in_node,
                         b->in_slot, val_ptr, vidx, pass_ptr, pidx, s.pass_node, s.pass_slot, ops, s.gather,
                         s.edge_index);
    }
  }
  // batches <= items; read back the batch table and the state sizes up to kCap entries each
  hipLaunchKernelGGL(k_typed_finish, dim3(16), dim3(kBlock), 0, st, err, meta, s.batch_depth, s.batch_op,
                     s.batch_rows, s.batch_goff, s.state_size, M, (int)nsize, kCap, tmp2.stage);
  if (hipGetLastError() != hipSuccess) return device_error("kernel launch failed");
  if (hipStreamSynchronize(st) != hipSuccess) return device_error("device error while scheduling");
  tmp1.waited = tmp2.waited = true;
  const int* hb = tmp2.stage;
  const int nb = M > 0 ? hb[2 + 4] : 0;
  s.nb = nb;
  if (nb <= kCap && (int)nsize <= kCap) {
    const int* hs = hb + kHdr;
    s.h_depth_b.assign(hs, hs + nb);
    s.h_op_b.assign(hs + kCap, hs + kCap + nb);
    s.h_rows_b.assign(hs + 2 * kCap, hs + 2 * kCap + nb);
    s.h_goff_b.assign(hs + 3 * kCap, hs + 3 * kCap + nb);
    s.h_state_size.assign(hs + 4 * kCap, hs + 4 * kCap + nsize);
  } else {
    std::vector<int>* dst[4] = {&s.h_depth_b, &s.h_op_b, &s.h_rows_b, &s.h_goff_b};
    const int* src[4] = {s.batch_depth, s.batch_op, s.batch_rows, s.batch_goff};
    bool ok = true;
    for (int k = 0; k < 4; ++k) {
      dst[k]->resize(nb);
      ok = ok && hipMemcpyAsync(dst[k]->data(), src[k], (size_t)nb * sizeof(int), hipMemcpyDeviceToHost, st) ==
                     hipSuccess;
    }
    s.h_state_size.resize(nsize);
    ok = ok && hipMemcpyAsync(s.h_state_size.data(), s.state_size, nsize * sizeof(int), hipMemcpyDeviceToHost, st) ==
                   hipSuccess;
    if (!ok || hipStreamSynchronize(st) != hipSuccess) return device_error("device error while reading the batches");
  }
  *out = h;
  return FOLD_OK;
}

}  // namespace fold
