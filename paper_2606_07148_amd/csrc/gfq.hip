// On-the-fly query support (Sec. V, GFQ): connected components by parallel
// union-find, edge updates on the resident graph, and the scoped answer.
#include "prim.h"

#include <algorithm>

#include "abcore_internal.h"
#include "wave.h"

namespace abc {

namespace {

__device__ __forceinline__ int32_t aload(const int32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void astore(int32_t *p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Union-find with parents that only ever point to smaller ids, so the root
// of every tree is the smallest id of its component (the canonical label).
// Reads are device-coherent atomics: a stale parent read could otherwise
// keep a thread retrying on an out-of-date root.
__device__ int32_t uf_find(int32_t *parent, int32_t x) {
  while (true) {
    const int32_t p = aload(&parent[x]);
    if (p == x) return x;
    const int32_t gp = aload(&parent[p]);
    if (gp == p) return p;
    astore(&parent[x], gp);  // path halving; gp is still an ancestor of x
    x = gp;
  }
}

// Ends also where both have one parent, without a look at the root: most calls
// find both ends in the largest tree, and once its root's line has been written
// in a launch, reads of it queue (2.7 ms of one relabelling of 5.5 M vertices).
__device__ void uf_union(int32_t *parent, int32_t a, int32_t b) {
  if (aload(&parent[a]) == aload(&parent[b])) return;
  while (true) {
    a = uf_find(parent, a);
    b = uf_find(parent, b);
    if (a == b) return;
    if (a > b) {
      int32_t t = a;
      a = b;
      b = t;
    }
    const int32_t old = atomicCAS(&parent[b], b, a);
    if (old == b) return;
    b = old;
  }
}

// The vertices a search for connected parts covers: those labelled `label`
// (all when it is negative; a row's live entries stay inside), or the members
// of a bitmap (a row's entries are tested too).
struct LabelScope {
  const int32_t *comp;
  int32_t label;
  __device__ __forceinline__ bool in(int64_t x) const { return label < 0 || comp[x] == label; }
  __device__ __forceinline__ bool near(int32_t w) const { return w >= 0; }
  // a vertex at or after sample i of k, or -1
  __device__ __forceinline__ int64_t sample(int i, int k, int64_t n) const {
    const int64_t x = (n * i) / k;
    return x < n && in(x) ? x : -1;
  }
};
struct MemberScope {
  const uint32_t *bits;
  __device__ __forceinline__ bool in(int64_t x) const { return (bits[x >> 5] >> (x & 31)) & 1u; }
  __device__ __forceinline__ bool near(int32_t w) const { return w >= 0 && in(w); }
  // (members may be few: the first one in the 64 words from the sample on)
  __device__ __forceinline__ int64_t sample(int i, int k, int64_t n) const {
    const int64_t words = (n + 31) / 32, w0 = (words * i) / k;
    for (int64_t w = w0; w < min(words, w0 + 64); ++w)
      if (bits[w] != 0) return 32 * w + (__ffs((int)bits[w]) - 1);
    return -1;
  }
};

// Hooking phase: the first unions, without an atomic.  Every lower vertex
// takes the first live entry of its row as parent (rows are ascending and
// upper ids precede lower ones: its smallest upper neighbour), then every
// upper vertex the smallest of the parents of its first kSampleLinks live
// entries, if smaller than itself.  Each thread writes only its own vertex's
// parent, and each parent is a smaller id of the same component, so the
// result is a forest for the union-find below; a hub's smallest neighbour
// has a very small id, so on skewed graphs almost every vertex ends in one
// tree.  (The Afforest strategy of Sutton, Ben-Nun and Barak, 2018, samples
// the first neighbours too, but unites them: here every neighbour of a hub
// then contended for the same few roots: a relabelling of 1.5 M vertices of
// 2e7 skewed edges took 2.3 to 5.2 ms by the graph's seed, all but 0.05 ms of
// it those unions; hooks and merges take 0.24 ms.)
constexpr int kSampleLinks = 2;
// Entries looked at for a live one; a vertex with none there stays a root.
constexpr int kHookProbe = 16;

template <class Scope>
__global__ void uf_hook_lower_kernel(const int64_t *__restrict__ off,
                                     const int32_t *__restrict__ cols, Scope scope,
                                     int32_t *parent, int64_t nU, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride) {
    if (!scope.in(x)) continue;
    int32_t p = (int32_t)x;
    if (x >= nU) {
      const int64_t s = off[x], e = min(off[x + 1], s + kHookProbe);
      for (int64_t j = s; j < e; ++j) {
        const int32_t w = cols[j];
        if (scope.near(w)) {
          p = w;
          break;
        }
      }
    }
    parent[x] = p;
  }
}

template <class Scope>
__global__ void uf_hook_upper_kernel(const int64_t *__restrict__ off,
                                     const int32_t *__restrict__ cols, Scope scope,
                                     int32_t *parent, int64_t nU) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < nU; x += stride) {
    if (!scope.in(x)) continue;
    int32_t p = (int32_t)x;
    const int64_t s = off[x], e = min(off[x + 1], s + kHookProbe);
    int links = 0;
    for (int64_t j = s; j < e && links < kSampleLinks; ++j) {
      const int32_t w = cols[j];
      if (!scope.near(w)) continue;
      p = min(p, parent[w]);  // a lower vertex's, final since the last launch
      ++links;
    }
    parent[x] = p;
  }
}

template <class Scope>
__global__ void uf_compress_kernel(int32_t *parent, Scope scope, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride)
    if (scope.in(x)) astore(&parent[x], uf_find(parent, (int32_t)x));
}

// Merging phase: the roots at the two ends of two more edges of every upper
// vertex, from the middle of its row, are joined by lowering the larger
// root's parent to the smaller root.  A minimum may overwrite another join,
// which is then not made: trees hold vertices of one component all the same,
// and the completion below walks every vertex outside the largest tree.  On
// 1.5 M vertices and 2e7 skewed edges the hooks leave 15,205 trees, the
// largest of 13% of the vertices, and a first launch two or one that hold
// 99% (90% and 9%, or 99%, by the seed): no join between two low roots need
// have been kept.  A second launch over every kMergeEvery-th vertex (kFind:
// roots looked up, since the trees are not compressed in between) joins
// those, and leaves 10,700 vertices of a few thousand entries outside.
//
// Nearly all joins lower one of a few dozen large roots, and same-address
// atomics (and stores) queue: each workgroup first takes the minimum per root
// in a small direct-mapped LDS table and adds each to memory once (a join
// whose slot another root holds goes to memory).  340 us without the table,
// 665 with plain stores in place of the minimum.
constexpr int kMergeBlock = 1024;
constexpr int kMergeSlots = 2048;
constexpr int kMergeEvery = 16;

template <bool kFind, class Scope>
__global__ __launch_bounds__(kMergeBlock) void uf_merge_kernel(
    const int64_t *__restrict__ off, const int32_t *__restrict__ cols, Scope scope,
    int32_t *parent, int64_t nU) {
  __shared__ int32_t key[kMergeSlots], low[kMergeSlots];
  for (int i = threadIdx.x; i < kMergeSlots; i += kMergeBlock) {
    key[i] = -1;
    low[i] = INT32_MAX;
  }
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * kMergeBlock;
  for (int64_t i = (int64_t)blockIdx.x * kMergeBlock + threadIdx.x;; i += stride) {
    const int64_t x = kFind ? i * kMergeEvery : i;
    if (x >= nU) break;
    if (!scope.in(x)) continue;
    const int64_t s = off[x], d = off[x + 1] - s;
    if (d == 0) continue;
    const int32_t w[2] = {cols[s + d / 3], cols[s + 2 * d / 3]};
    // (a parent lowered meanwhile may be read old or new: both are in the
    // vertex's component)
    const int32_t rx = kFind ? uf_find(parent, (int32_t)x) : parent[x];
    int32_t rw[2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
      rw[k] = !scope.near(w[k]) ? rx : kFind ? uf_find(parent, w[k]) : parent[w[k]];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int32_t lo = min(rx, rw[k]), hi = max(rx, rw[k]);
      if (lo == hi) continue;
      const int slot = (int)(((uint32_t)hi * 2654435761u) >> 21);
      static_assert(kMergeSlots == 1 << 11, "slot hash");
      int32_t held = __hip_atomic_load(&key[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (held < 0) {
        const int32_t old = atomicCAS(&key[slot], -1, hi);
        held = old < 0 ? hi : old;
      }
      if (held != hi)
        atomicMin(&parent[hi], lo);
      else if (__hip_atomic_load(&low[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > lo)
        atomicMin(&low[slot], lo);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kMergeSlots; i += kMergeBlock)
    if (key[i] >= 0) atomicMin(&parent[key[i]], low[i]);
}

// Every lower vertex unites with the first kSampleLinks entries of its row
// (sparse_merges, below).
template <class Scope>
__global__ void uf_sample_link_kernel(const int64_t *__restrict__ off,
                                      const int32_t *__restrict__ cols, Scope scope,
                                      int32_t *parent, int64_t nU, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = nU + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride) {
    if (!scope.in(x)) continue;
    const int64_t s = off[x], e = min(off[x + 1], s + kSampleLinks);
    for (int64_t j = s; j < e; ++j) {
      const int32_t w = cols[j];
      if (scope.near(w)) uf_union(parent, (int32_t)x, w);
    }
  }
}

// The most frequent root among kRootSamples evenly spaced vertices into
// *big (-1 when none of them is in scope): one workgroup, every thread
// counting its own sample among all of them in LDS, so that the choice
// needs no host.
constexpr int kRootSamples = 256;

template <class Scope>
__global__ __launch_bounds__(kRootSamples) void uf_big_root_kernel(const int32_t *parent,
                                                                   Scope scope, int64_t n,
                                                                   int32_t *big) {
  __shared__ __align__(16) int32_t roots[kRootSamples];
  __shared__ unsigned long long best;
  const int i = threadIdx.x;
  const int64_t x = scope.sample(i, kRootSamples, n);
  const int32_t mine = x >= 0 ? aload(&parent[x]) : -1;
  roots[i] = mine;
  if (i == 0) best = 0;
  __syncthreads();
  int c = 0;
  for (int j = 0; j < kRootSamples; j += 4) {
    const int4 r = *reinterpret_cast<const int4 *>(&roots[j]);
    c += (r.x == mine) + (r.y == mine) + (r.z == mine) + (r.w == mine);
  }
  // (the count in the high word decides, then the smaller root)
  if (mine >= 0)
    atomicMax(&best, ((unsigned long long)c << 32) | (uint32_t)(0x7FFFFFFF - mine));
  __syncthreads();
  if (i == 0) *big = best != 0 ? 0x7FFFFFFF - (int32_t)(uint32_t)best : -1;
}

// Completion: every vertex in scope outside the tree of root `big` unites
// with all of its neighbours (both layers' rows and inserted edges).  Edges
// with both ends in that tree need nothing: they are joined already.
template <class Scope>
__global__ __launch_bounds__(kBlock) void uf_rest_link_kernel(
    const int64_t *__restrict__ off, const int32_t *__restrict__ cols, Scope scope,
    int32_t *parent, const int32_t *ins_head, const int32_t *ins_next,
    const int32_t *ins_other, int64_t n, const int32_t *big_root) {
  const int32_t big = *big_root;
  const int gw = blockIdx.x * kWavesPerBlock + wave_in_block();
  const int nw = gridDim.x * kWavesPerBlock;
  for (int64_t b = (int64_t)gw * kWave; b < n; b += (int64_t)nw * kWave) {
    const int64_t xi = b + lane_id();
    int32_t x = -1;
    if (xi < n && scope.in(xi) && (big < 0 || uf_find(parent, (int32_t)xi) != big))
      x = (int32_t)xi;
    int64_t s = 0;
    int d = 0;
    if (x >= 0) {
      s = off[x];
      d = (int)(off[x + 1] - s);
    }
    const int incl = wave_incl_scan(d);
    const int total = __shfl(incl, kWave - 1, kWave);
    const int excl = incl - d;
    const int s_lo = (int)(uint32_t)(uint64_t)s;
    const int s_hi = (int)((uint64_t)s >> 32);
    for (int base = 0; base < total; base += kWave) {
      const int k = base + lane_id();
      const int kk = k < total ? k : total - 1;
      int j = 0;
#pragma unroll
      for (int step = 32; step > 0; step >>= 1) {
        int v = __shfl(incl, j + step - 1, kWave);
        if (v <= kk) j += step;
      }
      const int ex = __shfl(excl, j, kWave);
      const uint32_t lo32 = (uint32_t)__shfl(s_lo, j, kWave);
      const uint32_t hi32 = (uint32_t)__shfl(s_hi, j, kWave);
      const int32_t owner = __shfl(x, j, kWave);
      const int64_t start = (int64_t)(((uint64_t)hi32 << 32) | lo32);
      if (k < total) {
        const int32_t w = cols[start + (kk - ex)];
        if (scope.near(w)) uf_union(parent, owner, w);
      }
    }
    if (ins_head != nullptr && x >= 0) {
      for (int e = ins_head[x]; e >= 0; e = ins_next[e]) {
        const int32_t w = ins_other[e];
        if (scope.near(w)) uf_union(parent, x, w);
      }
    }
  }
}

__global__ void uf_label_kernel(int32_t *parent, int32_t *comp, int32_t label, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride)
    if (LabelScope{comp, label}.in(x)) comp[x] = uf_find(parent, (int32_t)x);
}

// The members in the trees of vx and vy (each only if a member itself) into
// bits, every word, and their number added to *count.
__global__ __launch_bounds__(kBlock) void uf_reached_kernel(const uint32_t *__restrict__ member,
                                                            int32_t *parent, int32_t vx,
                                                            int32_t vy, int64_t n,
                                                            uint32_t *__restrict__ bits,
                                                            int64_t nwords,
                                                            unsigned long long *count) {
  const MemberScope scope{member};
  // (a root is the vertex itself or smaller: -1 is no member's root)
  const int32_t r1 = scope.in(vx) ? uf_find(parent, vx) : -1;
  const int32_t r2 = scope.in(vy) ? uf_find(parent, vy) : -1;
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  unsigned long long c = 0;
  for (int64_t base = ((int64_t)blockIdx.x * kWavesPerBlock + wave_in_block()) * kWave;
       base < nwords * 32; base += stride) {
    const int64_t x = base + lane_id();
    bool p = false;
    if (x < n && scope.in(x)) {
      const int32_t r = uf_find(parent, (int32_t)x);
      p = r == r1 || r == r2;
    }
    const uint64_t mask = __ballot(p);
    const int64_t w0 = base / 32;
    if (lane_id() == 0) {
      bits[w0] = (uint32_t)mask;
      c += __popcll(mask);
    }
    if (lane_id() == 1 && w0 + 1 < nwords) bits[w0 + 1] = (uint32_t)(mask >> 32);
  }
  __shared__ unsigned long long s;
  if (threadIdx.x == 0) s = 0;
  __syncthreads();
  if (c != 0) atomicAdd(&s, c);
  __syncthreads();
  if (threadIdx.x == 0 && s != 0) atomicAdd(count, s);
}

__global__ void relabel_kernel(int32_t *comp, int64_t n, int32_t from, int32_t to) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride)
    if (comp[x] == from) comp[x] = to;
}

// The entry of y in row x and that of x in row y, by one wave (all lanes): a
// half of it searches each row, 32 probes to a step (a hub's row of 30,000 in
// four round trips; a thread's binary searches took 15 each).  Entries are
// read at device scope: an update before may have just changed them.
struct PairEntries {
  int64_t jx, jy;  // positions in cols, -1: not there
  bool live;       // the entry in row x is not deleted
};
__device__ __forceinline__ PairEntries find_pair(const int64_t *off, const int32_t *cols,
                                                 int32_t x, int32_t y) {
  const int l = lane_id() & 31;
  const bool second = lane_id() >= 32;
  const int32_t row = second ? y : x, key = second ? x : y;
  int64_t lo = off[row], hi = off[row + 1];
  auto half = [&](bool p) {
    const uint64_t m = __ballot(p);
    return (uint32_t)(second ? m >> 32 : m);
  };
  // entries before lo are below the key, those from hi on above it
  while (__ballot(hi - lo > 32)) {
    const int64_t len = hi - lo;
    const int64_t p = lo + len * (l + 1) / 33;
    bool below = false;
    if (len > 32) {
      const int32_t c = ld_agent(&cols[p]);
      below = (c < 0 ? ~c : c) < key;
    }
    const int before = __popc(half(below));
    if (len > 32) {
      const int64_t from = lo;
      if (before > 0) lo = from + len * before / 33 + 1;
      if (before < 32) hi = from + len * (before + 1) / 33 + 1;
    }
  }
  int32_t c = -1;
  bool here = false;
  if (lo + l < hi) {
    c = ld_agent(&cols[lo + l]);
    here = (c < 0 ? ~c : c) == key;
  }
  const uint32_t hit = half(here), live = half(here && c >= 0);
  const int64_t at = hit != 0 ? lo + __ffs((int)hit) - 1 : -1;
  PairEntries r;
  r.jx = __shfl((long long)at, 0, kWave);
  r.jy = __shfl((long long)at, 32, kWave);
  r.live = __shfl((int)live, 0, kWave) != 0;
  return r;
}

// What the host reads of an update (the same words of the pinned state).
struct UpdateResult {
  int32_t status, aux0, aux1;
};
static_assert(offsetof(PeelState, aux0) == offsetof(PeelState, status) + 4 &&
                  offsetof(PeelState, aux1) == offsetof(PeelState, status) + 8,
              "the result's words are the state's");

// Applies one update (one thread).  Validation precedes every write,
// so a rejected update leaves the graph untouched.  st->status: 0 applied,
// 1 applied using the new delta slot `slot`, -5 present (insertion),
// -4 absent (deletion).  aux0/aux1 receive the labels of u and v before the
// update.
__device__ void apply_update(const int64_t *off, int32_t *cols, int32_t *deg0,
                             const int32_t *comp, int32_t *ins_head, int32_t *ins_next,
                             int32_t *ins_other, int64_t slot, int32_t nU, int32_t u, int32_t v,
                             int32_t op, UpdateResult *st) {
  const int32_t x = u, y = nU + v;
  // base CSR entry of the pair (row x holds y, row y holds x)
  const PairEntries pair = find_pair(off, cols, x, y);
  if (lane_id() != 0) return;
  const int64_t jx = pair.jx, jy = pair.jy;
  const bool csr_live = jx >= 0 && pair.live;
  st->aux0 = comp != nullptr ? comp[x] : -1;
  st->aux1 = comp != nullptr ? comp[y] : -1;
  // inserted half-edge of the pair in row x (live or deleted)
  int32_t ex = -1;
  for (int32_t e = ins_head != nullptr ? ins_head[x] : -1; e >= 0; e = ins_next[e]) {
    const int32_t o = ins_other[e];
    if ((o < 0 ? ~o : o) == y) {
      ex = e;
      break;
    }
  }
  const bool delta_live = ex >= 0 && ins_other[ex] >= 0;
  const bool present = csr_live || delta_live;
  if (op > 0) {
    if (present) {
      st->status = -(int32_t)ABCORE_EEXIST;
      return;
    }
    if (jx >= 0) {  // revive the tombstoned CSR pair
      cols[jx] = y;
      cols[jy] = x;
      st->status = 0;
    } else if (ex >= 0) {  // revive the deleted inserted pair
      ins_other[ex] = y;
      ins_other[ex ^ 1] = x;
      st->status = 0;
    } else {
      const int32_t hx = (int32_t)(2 * slot), hy = (int32_t)(2 * slot + 1);
      ins_other[hx] = y;
      ins_other[hy] = x;
      ins_next[hx] = ins_head[x];
      ins_head[x] = hx;
      ins_next[hy] = ins_head[y];
      ins_head[y] = hy;
      st->status = 1;
    }
    deg0[x] += 1;
    deg0[y] += 1;
  } else {
    if (!present) {
      st->status = -(int32_t)ABCORE_ENOENT;
      return;
    }
    if (csr_live) {
      cols[jx] = ~y;
      cols[jy] = ~x;
    } else {
      ins_other[ex] = ~y;
      ins_other[ex ^ 1] = ~x;
    }
    deg0[x] -= 1;
    deg0[y] -= 1;
    st->status = 0;
  }
}

// The update (thread 0), and after a deletion on exact labels (settle) the
// common cases in which it splits nothing that needs a search: an endpoint
// left without edges becomes its own component (unless it was the label of
// vertices that stay), and endpoints still joined by a path of length three
// x - v' - u' - y leave every label as it is.  status 2: the labels are
// settled; 0: the component has to be labelled again (0.24 ms at 1.5 M
// vertices, and growing with them).  The path is looked for in bounded work,
// so not finding one proves nothing: the first kSettleRow entries of x's row
// in LDS, against the first kSettleScan entries of the rows of the first
// kSettleCand neighbours of y, one row per wave at a time.  Inserted edges
// take no part.  Measured at 2e7 edges: 11 us with the path found, against
// 5 us for the update alone.
constexpr int kSettleBlock = 1024;
constexpr int kSettleRow = 8192;
constexpr int kSettleCand = 64;
constexpr int kSettleScan = 1024;

__global__ __launch_bounds__(kSettleBlock) void update_kernel(
    const int64_t *off, int32_t *cols, int32_t *deg0, int32_t *comp, int32_t *ins_head,
    int32_t *ins_next, int32_t *ins_other, int64_t slot, int32_t nU, int32_t u, int32_t v,
    int32_t op, int settle, UpdateResult *out) {
  __shared__ int32_t row[kSettleRow];
  __shared__ int s_found;
  __shared__ UpdateResult s_res;
  UpdateResult *st = &s_res;
  if (threadIdx.x == 0) s_found = 0;
  if (wave_in_block() == 0)
    apply_update(off, cols, deg0, comp, ins_head, ins_next, ins_other, slot, nU, u, v, op, st);
  // the result, to host-visible memory (a copy of the state took 4 us more)
  auto publish = [&]() {
    if (threadIdx.x != 0) return;
    const int32_t v[3] = {s_res.status, s_res.aux0, s_res.aux1};
    int32_t *to = &out->status;
    for (int i = 0; i < 3; ++i)
      __hip_atomic_store(to + i, v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  };
  if (op > 0 || !settle) {
    publish();
    return;
  }
  __syncthreads();  // the deletion is visible to the workgroup
  if (st->status != 0) {
    publish();
    return;
  }
  const int32_t x = u, y = nU + v;
  const int32_t dx = deg0[x], dy = deg0[y];
  __syncthreads();  // (status is rewritten below)
  if (dx == 0 || dy == 0) {
    if (threadIdx.x != 0) return;
    // y, a lower vertex, labels no vertex but itself
    if (dy == 0) comp[y] = y;
    if (dy == 0 || comp[x] != x) {
      if (dx == 0) comp[x] = x;
      st->status = 2;
    }
    publish();
    return;
  }
  const int64_t xa = off[x];
  const int nrow = (int)min(off[x + 1] - xa, (int64_t)kSettleRow);
  for (int i = threadIdx.x; i < nrow; i += kSettleBlock) row[i] = cols[xa + i];
  __syncthreads();
  const int64_t ya = off[y];
  const int ncand = (int)min(off[y + 1] - ya, (int64_t)kSettleCand);
  for (int c = wave_in_block(); c < ncand; c += kSettleBlock / kWave) {
    if (__hip_atomic_load(&s_found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) break;
    const int32_t w = cols[ya + c];
    if (w < 0) continue;  // deleted, x among them
    const int64_t ra = off[w], rb = min(off[w + 1], ra + kSettleScan);
    for (int64_t j0 = ra; j0 < rb; j0 += kWave) {
      const int64_t j = j0 + lane_id();
      const int32_t z = j < rb ? cols[j] : -1;
      bool hit = false;
      if (z >= 0) {
        // rows are ascending once tombstones ~c are decoded
        int lo = 0, hi = nrow;
        while (lo < hi) {
          const int mid = (lo + hi) / 2;
          const int32_t r = row[mid];
          if ((r < 0 ? ~r : r) < z)
            lo = mid + 1;
          else
            hi = mid;
        }
        hit = lo < nrow && row[lo] == z;
      }
      if (__ballot(hit)) {
        if (lane_id() == 0)
          __hip_atomic_store(&s_found, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        break;
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && s_found) st->status = 2;
  publish();
}

// A window of served updates, applied in order by a single wave (the order
// of the stream: each update is validated against the graph after the
// previous ones).  Append-only, so that queries of earlier versions still
// peeling see their own graph: a deleted base entry gets its deletion
// version in del_ver before it is tombstoned, a deleted inserted pair in
// pair_del_ver, and an insertion always takes a new pair (pairs are
// numbered in insertion order; a query sees pairs below its limit).  Each
// record: status (0, -EEXIST, -ENOENT), version (valid updates count up from
// ver_base), pairs after the update, labels of the endpoints before the
// window.  The updates arrive with the launch and
// the records go to pinned host memory (the copies took longer than the
// kernel).
__global__ void update_window_kernel(const int64_t *off, int32_t *cols, int32_t *deg0,
                                     const int32_t *comp, int32_t *ins_head, int32_t *ins_next,
                                     int32_t *ins_other, int32_t *del_ver,
                                     int32_t *pair_del_ver, int32_t pair_base,
                                     int32_t ver_base, int32_t nU, WindowUpdates upd, int w,
                                     WindowRecord *rec) {
  int32_t ver = ver_base, pairs = pair_base;
  for (int i = 0; i < w; ++i) {
    const int32_t x = upd.v[3 * i], y = nU + upd.v[3 * i + 1], op = upd.v[3 * i + 2];
    const PairEntries pair = find_pair(off, cols, x, y);
    // the update itself by the first lane; its stores are done before the
    // next search
    if (lane_id() != 0) continue;
    WindowRecord r;
    r.label_u = comp[x];
    r.label_v = comp[y];
    const int64_t jx = pair.jx, jy = pair.jy;
    const bool csr_live = jx >= 0 && pair.live;
    int32_t ex = -1;  // live inserted half-edge of the pair in row x
    for (int32_t e = pairs > 0 ? ins_head[x] : -1; e >= 0; e = ins_next[e])
      if (ins_other[e] == y) {
        ex = e;
        break;
      }
    const bool present = csr_live || ex >= 0;
    r.status = 0;
    r.version = -1;
    if (op > 0 && present) {
      r.status = -(int32_t)ABCORE_EEXIST;
    } else if (op < 0 && !present) {
      r.status = -(int32_t)ABCORE_ENOENT;
    } else if (op > 0) {
      const int32_t v = ++ver;
      const int32_t hx = 2 * pairs, hy = 2 * pairs + 1;
      ins_other[hx] = y;
      ins_other[hy] = x;
      pair_del_ver[pairs] = 0x7FFFFFFF;
      ins_next[hx] = ins_head[x];
      ins_next[hy] = ins_head[y];
      __threadfence();  // the pair is complete before the lists point to it
      astore(&ins_head[x], hx);
      astore(&ins_head[y], hy);
      ++pairs;
      deg0[x] += 1;
      deg0[y] += 1;
      r.version = v;
    } else {
      const int32_t v = ++ver;
      if (csr_live) {
        del_ver[jx] = v;
        del_ver[jy] = v;
        __threadfence();  // the version is visible before the tombstone
        astore(&cols[jx], ~y);
        astore(&cols[jy], ~x);
      } else {
        pair_del_ver[ex >> 1] = v;
        __threadfence();
        astore(&ins_other[ex], ~y);
        astore(&ins_other[ex ^ 1], ~x);
      }
      deg0[x] -= 1;
      deg0[y] -= 1;
      r.version = v;
    }
    r.pairs_after = pairs;
    rec[i] = r;
    // (relaxed device-scope stores and loads: a wait orders them, where a
    // fence would write back the L2)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
  }
}

// Membership of the two endpoints after the scoped peel.
__global__ void answer_kernel(const int32_t *deg, int32_t x, int32_t y, int32_t thrU,
                              int32_t thrL, PeelState *st) {
  const int32_t bits = (deg[x] >= thrU ? 1 : 0) | (deg[y] >= thrL ? 2 : 0);
  st->aux0 = bits;
}

// Current-graph CSR export, rows ascending: live base entries merged with
// the live inserted ones.  Rows that the updates left alone (full degree, no
// inserted list) are copied, 64 rows of at most kPiece entries or 64 pieces
// of longer rows per wave, entry by entry across the lanes whatever the
// degree mix: an entry moves by one shift per row.  The other rows follow one
// per wave: an entry's position is the live entries before it (ballots) plus
// the inserted ones below it (a short list in LDS).  (A thread per row copied
// hubs of 50,000 entries serially, 8.7 ms at 2e7 edges.)
constexpr int kExportIns = 64;  // inserted entries of a row held in LDS

// Copies d entries from s to s + shift (per lane; d <= kPiece).
__device__ __forceinline__ void copy_rows(const int32_t *__restrict__ cols,
                                          int32_t *__restrict__ out, int64_t s, int d,
                                          int64_t shift) {
  constexpr int kU = 4;  // copies in flight per lane
  const int incl = wave_incl_scan(d);
  const int total = __shfl(incl, kWave - 1, kWave);
  const int64_t from = s - (incl - d);  // position of the batch's entry 0, by this row
  for (int base = 0; base < total; base += kU * kWave) {
    int32_t w[kU];
    int64_t to[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int k = base + u * kWave + lane_id();
      const int kk = min(k, total - 1);
      int j = 0;
#pragma unroll
      for (int step = 32; step > 0; step >>= 1)
        if (__shfl(incl, j + step - 1, kWave) <= kk) j += step;
      const int64_t pos = __shfl(from, j, kWave) + kk;
      to[u] = pos + __shfl(shift, j, kWave);
      w[u] = cols[pos];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (base + u * kWave + lane_id() < total) out[to[u]] = w[u];
  }
}

// One changed row: base entries [s, s + d), output from o0; ins (kExportIns
// ints of LDS) and the wave are its own.
__device__ __forceinline__ void export_changed_row(const int32_t *__restrict__ cols, int64_t s,
                                                   int64_t d, int head,
                                                   const int32_t *__restrict__ ins_next,
                                                   const int32_t *__restrict__ ins_other,
                                                   int64_t o0, int32_t *__restrict__ out,
                                                   int32_t *ins) {
  constexpr int kU = 4;
  int all = 0;
  if (lane_id() == 0) {
    // the live inserted entries, ascending; a list that does not fit is
    // merged entry by entry below
    for (int e = head; e >= 0; e = ins_next[e]) {
      const int32_t v = ins_other[e];
      if (v < 0) continue;
      if (all < kExportIns) {
        int p = all;
        while (p > 0 && ins[p - 1] > v) {
          ins[p] = ins[p - 1];
          --p;
        }
        ins[p] = v;
      }
      ++all;
    }
  }
  all = __shfl(all, 0, kWave);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int c = all <= kExportIns ? all : 0;
  int64_t live = 0, before = 0;  // before: live entries below lane i's inserted one
  for (int64_t k0 = 0; k0 < d; k0 += kU * kWave) {
    int32_t w[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t k = k0 + u * kWave + lane_id();
      w[u] = k < d ? cols[s + k] : -1;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint64_t mask = __ballot(w[u] >= 0);
      int below = 0;
      for (int i = 0; i < c; ++i) {
        const bool less = w[u] >= 0 && w[u] < ins[i];
        if (!less && w[u] >= 0) ++below;
        const int cnt = __popcll(__ballot(less));
        if (lane_id() == i) before += cnt;
      }
      if (w[u] >= 0) out[o0 + live + __popcll(mask & lanemask_lt()) + below] = w[u];
      live += __popcll(mask);
    }
  }
  if (lane_id() < c) out[o0 + before + lane_id()] = ins[lane_id()];
  if (all > kExportIns && lane_id() == 0) {
    int64_t o = o0 + live;
    for (int e = head; e >= 0; e = ins_next[e]) {
      const int32_t v = ins_other[e];
      if (v < 0) continue;
      int64_t p = o++;
      while (p > o0 && out[p - 1] > v) {
        out[p] = out[p - 1];
        --p;
      }
      out[p] = v;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(kBlock) void export_rows_kernel(
    const int64_t *__restrict__ off, const int32_t *__restrict__ cols,
    const int32_t *__restrict__ deg0, const int32_t *__restrict__ ins_head,
    const int32_t *__restrict__ ins_next, const int32_t *__restrict__ ins_other,
    const int32_t *__restrict__ piece_row, const int64_t *__restrict__ piece_start,
    const int64_t *__restrict__ out_off, int32_t *__restrict__ out_cols, int64_t n,
    int64_t npieces) {
  __shared__ int32_t s_ins[kWavesPerBlock][kExportIns];
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + wave_in_block();
  const int64_t nw = (int64_t)gridDim.x * kWavesPerBlock;
  auto unchanged = [&](int64_t x, int64_t d) {
    return deg0[x] == d && (ins_head == nullptr || ins_head[x] < 0);
  };
  for (int64_t b = gw * kWave; b < n; b += nw * kWave) {
    const int64_t x = b + lane_id();
    int64_t s = 0, shift = 0, d = 0;
    bool same = true;
    if (x < n) {
      s = off[x];
      d = off[x + 1] - s;
      shift = out_off[x] - s;
      same = unchanged(x, d);
    }
    copy_rows(cols, out_cols, s, same && d <= kPiece ? (int)d : 0, shift);
    for (uint64_t rows = __ballot(!same); rows != 0; rows &= rows - 1) {
      const int j = __ffsll((unsigned long long)rows) - 1;
      const int64_t rs = __shfl(s, j, kWave);
      export_changed_row(cols, rs, __shfl(d, j, kWave),
                         ins_head != nullptr ? ins_head[b + j] : -1, ins_next, ins_other,
                         rs + __shfl(shift, j, kWave), out_cols, s_ins[wave_in_block()]);
    }
  }
  for (int64_t b = gw * kWave; b < npieces; b += nw * kWave) {
    const int64_t p = b + lane_id();
    int64_t s = 0, shift = 0;
    int d = 0;
    if (p < npieces) {
      const int32_t x = piece_row[p];
      s = piece_start[p];
      const int64_t rs = off[x], re = off[x + 1];
      shift = out_off[x] - rs;
      if (unchanged(x, re - rs)) d = (int)(min(s + kPiece, re) - s);
    }
    copy_rows(cols, out_cols, s, d, shift);
  }
}

__global__ void widen_deg_kernel(const int32_t *deg, int64_t n, int64_t *out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += stride)
    out[i] = i < n ? (int64_t)deg[i] : 0;
}

int small_grid(const Graph &g, int64_t items) {
  return (int)std::max<int64_t>(1, std::min<int64_t>((items + 255) / 256, g.cu_count * 8));
}

}  // namespace

// The forest of connected parts of a scope in g.parent: vertices of one part
// have one root, the smallest id in it.  Stream-ordered; the root of the
// largest tree sits in the partial-sum buffer (reset before every
// computation).  merges (sparse graphs): that many launches of the merging
// phase, the trees compressed after each, then unions of the lower vertices'
// first entries; 0: as the merging phase describes.
template <class Scope>
static void launch_parts(Graph &g, Scope scope, int merges, hipStream_t s) {
  const int32_t *head = g.delta.count > 0 ? g.delta.head : nullptr;
  int32_t *d_big = reinterpret_cast<int32_t *>(g.part);
  uf_hook_lower_kernel<<<small_grid(g, g.n), 256, 0, s>>>(g.off, g.cols, scope, g.parent, g.nU,
                                                          g.n);
  uf_hook_upper_kernel<<<small_grid(g, g.nU), 256, 0, s>>>(g.off, g.cols, scope, g.parent, g.nU);
  uf_compress_kernel<<<small_grid(g, g.n), 256, 0, s>>>(g.parent, scope, g.n);
  auto merge_grid = [&](int64_t items) {
    return (int)std::max<int64_t>(
        1, std::min<int64_t>((items + kMergeBlock - 1) / kMergeBlock, g.cu_count));
  };
  for (int i = 0; i < std::max(merges, 1); ++i) {
    uf_merge_kernel<false><<<merge_grid(g.nU), kMergeBlock, 0, s>>>(g.off, g.cols, scope,
                                                                    g.parent, g.nU);
    if (merges > 0) uf_compress_kernel<<<small_grid(g, g.n), 256, 0, s>>>(g.parent, scope, g.n);
  }
  if (merges > 0)
    uf_sample_link_kernel<<<small_grid(g, g.nL), 256, 0, s>>>(g.off, g.cols, scope, g.parent,
                                                              g.nU, g.n);
  else
    uf_merge_kernel<true><<<merge_grid(g.nU / kMergeEvery + 1), kMergeBlock, 0, s>>>(
        g.off, g.cols, scope, g.parent, g.nU);
  uf_compress_kernel<<<small_grid(g, g.n), 256, 0, s>>>(g.parent, scope, g.n);
  uf_big_root_kernel<<<1, kRootSamples, 0, s>>>(g.parent, scope, g.n, d_big);
  uf_rest_link_kernel<<<wide_grid(g), kBlock, 0, s>>>(g.off, g.cols, scope, g.parent, head,
                                                      g.delta.next, g.delta.other, g.n, d_big);
}

// Launches of the merging phase where few edges and no hubs leave the hooks
// many small trees, whose joining in the completion is slow: medians over
// uniform graphs, one merge and the strided one / three merges and the unions:
// 100,000 vertices with 95,000 edges 0.49 / 0.17 ms, 2 M with 2.1 M 1.2 / 0.73,
// 5.5 M with 6.3 M 1.3 / 1.0; a random tree of 2 M 3.8 / 2.7, a path of 2 M 3.6 /
// 0.75, of 200,000 0.33 / 0.47.  With fewer than half an edge a vertex (0.46 / 0.66
// at 5.5 M and 0.4), more than 7/4 (0.40 / 0.45 at 2 M and 2), long rows (0.28 for
// both at 1.5 M and 0.8) or more vertices (1.9 / 2.6 at 18 M and 1.1) the general
// merging is the faster, or the same.
static int sparse_merges(const Graph &g) {
  const int64_t n = g.n, m = g.m_csr;
  return g.nheavy == 0 && n <= (8 << 20) && 2 * m > n && 4 * m <= 7 * n ? 3 : 0;
}

// Component labels for the whole graph (label < 0) or re-labelling of the
// vertices currently labelled `label` (deletion may split that component).
hipError_t launch_cc(Graph &g, int32_t label, hipStream_t s) {
  launch_parts(g, LabelScope{g.comp, label}, sparse_merges(g), s);
  uf_label_kernel<<<small_grid(g, g.n), 256, 0, s>>>(g.parent, g.comp, label, g.n);
  return hipGetLastError();
}

// The members (a bitmap) connected to vx or vy through members.  One forest of
// all members' parts: a fixed number of launches, whatever the distances.
hipError_t launch_reached(Graph &g, const uint32_t *member, int32_t vx, int32_t vy,
                          uint32_t *bits, unsigned long long *count, hipStream_t s) {
  const int64_t nwords = (g.n + 31) / 32;
  launch_parts(g, MemberScope{member}, 0, s);
  uf_reached_kernel<<<small_grid(g, g.n), kBlock, 0, s>>>(member, g.parent, vx, vy, g.n, bits,
                                                          nwords, count);
  return hipGetLastError();
}

hipError_t launch_relabel(Graph &g, int32_t from, int32_t to, hipStream_t s) {
  relabel_kernel<<<small_grid(g, g.n), 256, 0, s>>>(g.comp, g.n, from, to);
  return hipGetLastError();
}

hipError_t launch_update(Graph &g, int32_t u, int32_t v, int32_t op, int64_t slot,
                         hipStream_t s) {
  const bool settle = op < 0 && g.comp_valid && g.comp_exact;
  update_kernel<<<1, settle ? kSettleBlock : kWave, 0, s>>>(
      g.off, g.cols, g.deg0, g.comp_valid ? g.comp : nullptr, g.delta.head, g.delta.next,
      g.delta.other, slot, g.nU, u, v, op, settle ? 1 : 0,
      reinterpret_cast<UpdateResult *>(&g.h_state->status));
  return hipGetLastError();
}

hipError_t launch_answer(Graph &g, int32_t x, int32_t y, int32_t thrU, int32_t thrL,
                         hipStream_t s) {
  answer_kernel<<<1, 1, 0, s>>>(g.deg, x, y, thrU, thrL, g.state);
  return hipGetLastError();
}

hipError_t launch_update_window(Graph &g, const WindowUpdates &upd, int w, WindowRecord *rec,
                                hipStream_t s) {
  update_window_kernel<<<1, kWave, 0, s>>>(g.off, g.cols, g.deg0, g.comp, g.delta.head,
                                       g.delta.next, g.delta.other, g.del_ver, g.pair_del_ver,
                                       (int32_t)g.delta.count, g.upd_version, g.nU, upd, w,
                                           rec);
  return hipGetLastError();
}

// Writes the current CSR (n+1 offsets, 2m entries) to caller buffers: on a
// graph unchanged since its build the handle's own arrays (0.06 ms at 2e7
// edges), else the rows with their updates.
hipError_t launch_export(Graph &g, int64_t *out_off, int32_t *out_cols, hipStream_t s) {
  if (g.version == 0 && g.delta.count == 0) {
    hipError_t e = hipMemcpyAsync(out_off, g.off, sizeof(int64_t) * (g.n + 1),
                                  hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess && out_cols != nullptr && g.m_csr > 0)
      e = hipMemcpyAsync(out_cols, g.cols, sizeof(int32_t) * 2 * g.m_csr,
                         hipMemcpyDeviceToDevice, s);
    return e == hipSuccess ? hipStreamSynchronize(s) : e;
  }
  int64_t *tmp64 = nullptr;
  void *temp = nullptr;
  size_t temp_bytes = 0;
  hipError_t e = dev_malloc_async(&tmp64, sizeof(int64_t) * (g.n + 1), s);
  if (e != hipSuccess) return e;
  widen_deg_kernel<<<small_grid(g, g.n + 1), 256, 0, s>>>(g.deg0, g.n, tmp64);
  e = prim::exclusive_sum(nullptr, temp_bytes, tmp64, out_off, (size_t)(g.n + 1), s);
  if (e == hipSuccess) e = dev_malloc_async(&temp, std::max<size_t>(temp_bytes, 16), s);
  if (e == hipSuccess)
    e = prim::exclusive_sum(temp, temp_bytes, tmp64, out_off, (size_t)(g.n + 1), s);
  if (e == hipSuccess && out_cols != nullptr) {
    const int32_t *head = g.delta.count > 0 ? g.delta.head : nullptr;
    export_rows_kernel<<<wide_grid(g), kBlock, 0, s>>>(
        g.off, g.cols, g.deg0, head, g.delta.next, g.delta.other, g.piece_row, g.piece_start,
        out_off, out_cols, g.n, g.npieces);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (temp) (void)dev_free_async(temp, s);
  (void)dev_free_async(tmp64, s);
  return e;
}

}  // namespace abc
