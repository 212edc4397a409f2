// (alpha,beta)-cores of graphs that fit one workgroup's LDS: a query is a
// single launch of a single workgroup (a batch: a workgroup per query).
//
// Both algorithms give the same core: a GCC+ query between unequal thresholds
// (43 us by classification) runs the same peel once the core numbers are there.
//
// On a graph of a few thousand vertices the scan, the first round and the
// peel take three launches of a worklist spread over the whole chip, whose
// handshakes through memory are all the time there is (38 us for 20,000 edges
// on 3,500 vertices).  Here the degrees, the row starts and the worklist live
// in LDS: a hop costs one load of neighbours and an LDS atomic, a round two
// barriers (8 us for the same).  What bounds it is that chain, and one compute
// unit's loads when much of the graph falls.
#include "abcore_internal.h"
#include "wave.h"

namespace abc {

constexpr int kTinyBlock = 1024;
constexpr int kTinyLanes = 8;    // lanes that walk one piece of a row
constexpr int kTinyPiece = 32;   // entries of a piece
constexpr int kTinyLoads = kTinyPiece / kTinyLanes;
constexpr int kTinyGroups = kTinyBlock / kTinyLanes;

// Rows are queued in pieces, an item being its first entry and its length
// (6 bits), so one long row is walked by as many lanes as several short ones.
constexpr int kTinyLenBits = 6;

// Entries of the largest graph of which single queries run this way.  One
// compute unit walks about 2 G entries/s of short rows, so a query near the
// mean degree, that removes nearly everything in rounds, takes 28 us here and
// 46 in the general path at 40,000 entries, 39 and 61 at 80,000, but 66 and
// 48 at 130,000 (9.6 and 34 us where little falls).  The queries of a batch
// run side by side: four times as many entries with four of them.
constexpr int64_t kTinyEntries = 5 << 14;

static int64_t tiny_items(const Graph &g) { return g.n + 2 * g.m_csr / kTinyPiece; }
static size_t tiny_lds(const Graph &g) {
  return sizeof(int32_t) * (size_t)(2 * g.n + 1 + tiny_items(g) + g.n / 32 + 2);
}

__global__ __launch_bounds__(kTinyBlock) void tiny_kernel(const int64_t *__restrict__ off,
                                                          const int32_t *__restrict__ cols,
                                                          const int32_t *__restrict__ deg0,
                                                          int32_t n, int32_t nU, int32_t nitems,
                                                          TinyQueries queries,
                                                          uint32_t *__restrict__ bits) {
  extern __shared__ int32_t s_tiny[];
  __shared__ int s_tail, s_f0;
  int32_t *deg = s_tiny;
  uint32_t *start = reinterpret_cast<uint32_t *>(s_tiny + n);  // n + 1 row starts
  uint32_t *item = start + n + 1;
  uint32_t *alive = item + nitems;  // the scan's survivors, a bit each
  const int32_t thrU = queries.thrU[blockIdx.x], thrL = queries.thrL[blockIdx.x];
  const int nwords = (n + 31) / 32;
  bits += (int64_t)blockIdx.x * nwords;
  if (threadIdx.x == 0) s_tail = s_f0 = 0;
  for (int x = threadIdx.x; x <= n; x += kTinyBlock) {
    start[x] = (uint32_t)off[x];
    if (x < n) deg[x] = deg0[x];
  }
  __syncthreads();
  const int total = (int)start[n];
  auto below = [&](int x) { return deg[x] < (x < nU ? thrU : thrL); };
  // the pieces of a row from slot `at` on (a vertex is queued once)
  auto put = [&](uint32_t s, int d, int at) {
    for (int i = 0; i < d; i += kTinyPiece)
      item[at++] = ((s + (uint32_t)i) << kTinyLenBits) | (uint32_t)min(d - i, kTinyPiece);
  };
  // queues the rows of the vertices that pass; returns this lane's entries
  auto queue_rows = [&](auto pass) {
    int entries = 0;
    for (int b = wave_in_block() * kWave; b < n; b += kTinyBlock) {
      const int x = b + lane_id();
      uint32_t s = 0;
      int d = 0;
      if (x < n && pass(x)) {
        s = start[x];
        d = (int)(start[x + 1] - s);
      }
      entries += d;
      const int pieces = (d + kTinyPiece - 1) / kTinyPiece;
      const int upto = wave_incl_scan(pieces);
      int base = 0;
      if (lane_id() == kWave - 1 && upto > 0) base = atomicAdd(&s_tail, upto);
      put(s, d, __shfl(base, kWave - 1, kWave) + upto - pieces);
    }
    return entries;
  };
  // calls use(item, entries) for the items from lo to hi, kTinyLanes lanes each
  const int lane = threadIdx.x % kTinyLanes;
  auto walk = [&](int lo, int hi, auto use) {
    for (int i = lo + (int)threadIdx.x / kTinyLanes; i < hi; i += kTinyGroups) {
      const uint32_t s = item[i] >> kTinyLenBits;
      const int d = (int)(item[i] & ((1u << kTinyLenBits) - 1u));
      int32_t w[kTinyLoads];
#pragma unroll
      for (int u = 0; u < kTinyLoads; ++u) {
        const int k = u * kTinyLanes + lane;
        w[u] = k < d ? cols[s + (uint32_t)k] : -1;  // (deleted entries are negative)
      }
      use(i, w);
    }
  };
  const int f0 = wave_sum(queue_rows(below));
  if (lane_id() == 0 && f0 > 0) atomicAdd(&s_f0, f0);
  __syncthreads();
  if (2 * (int64_t)s_f0 > total) {
    // the survivors have fewer entries than the scan's frontier: they count
    // their neighbours in it, and those that fall start the worklist
    for (int b = wave_in_block() * kWave; b < n; b += kTinyBlock) {
      const int x = b + lane_id();
      const uint64_t mask = __ballot(x < n && !below(x));
      if (lane_id() == 0) alive[b / 32] = (uint32_t)mask;
      if (lane_id() == 1 && b + 32 < n) alive[b / 32 + 1] = (uint32_t)(mask >> 32);
    }
    if (threadIdx.x == 0) s_tail = 0;
    __syncthreads();
    auto survives = [&](int x) { return ((alive[x >> 5] >> (x & 31)) & 1u) != 0; };
    queue_rows(survives);
    __syncthreads();
    walk(0, s_tail, [&](int i, const int32_t (&w)[kTinyLoads]) {
      int gone = 0;
#pragma unroll
      for (int u = 0; u < kTinyLoads; ++u) gone += w[u] >= 0 && !survives(w[u]) ? 1 : 0;
      if (gone == 0) return;
      // the row of the piece: the last one that starts at or before it (rows
      // without entries start where the next one does)
      const uint32_t s = item[i] >> kTinyLenBits;
      int x = 0;
      for (int end = n; end - x > 1;) {
        const int mid = (x + end) / 2;
        if (start[mid] <= s)
          x = mid;
        else
          end = mid;
      }
      atomicSub(&deg[x], gone);
    });
    __syncthreads();
    if (threadIdx.x == 0) s_tail = 0;
    __syncthreads();
    queue_rows([&](int x) { return survives(x) && below(x); });
  }
  for (int lo = 0;;) {
    __syncthreads();
    const int hi = s_tail;
    __syncthreads();  // (every thread has read it before the round appends)
    if (hi == lo) break;
    walk(lo, hi, [&](int, const int32_t (&w)[kTinyLoads]) {
      int32_t old[kTinyLoads];
#pragma unroll
      for (int u = 0; u < kTinyLoads; ++u)
        old[u] = w[u] >= 0 ? atomicSub(&deg[w[u]], 1) : INT32_MIN;
#pragma unroll
      for (int u = 0; u < kTinyLoads; ++u) {
        const int32_t x = w[u];
        // the decrement from the threshold queues x (one thread's)
        if (old[u] != (x < nU ? thrU : thrL)) continue;
        const uint32_t s = start[x];
        const int d = (int)(start[x + 1] - s);
        put(s, d, atomicAdd(&s_tail, (d + kTinyPiece - 1) / kTinyPiece));
      }
    });
    lo = hi;
  }
  for (int b = wave_in_block() * kWave; b < nwords * 32; b += kTinyBlock) {
    const int x = b + lane_id();
    const uint64_t mask = __ballot(x < n && deg[x] >= (x < nU ? thrU : thrL));
    const int w = b / 32;
    if (lane_id() == 0) bits[w] = (uint32_t)mask;
    if (lane_id() == 1 && w + 1 < nwords) bits[w + 1] = (uint32_t)(mask >> 32);
  }
}

// Whether `count` queries of this handle run in one workgroup each: the graph fits,
// nothing was inserted since the build (inserted edges are chained outside
// the rows) and every option that names another mapping is at its default.
bool tiny_ready(const Graph &g, int32_t count) {
  return g.n > 0 && 2 * g.m_csr <= kTinyEntries * std::min(count, 4) &&
         tiny_lds(g) + 1024 <= g.lds_per_block &&
         g.delta.count == 0 && g.peel_mode == 3 && g.pull_mode == 0 && !g.tuned &&
         g.append_sub < 0 && g.spin_limit == 0 && g.dbg_enqueue == nullptr;
}

hipError_t prepare_tiny_kernel(Graph &g) {
  if (tiny_lds(g) + 1024 > g.lds_per_block) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void *>(&tiny_kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)g.lds_per_block - 1024);
}

// The cores of `count` queries, query i's into bits + i * ceil(n / 32).
hipError_t launch_tiny(Graph &g, const int32_t *thrU, const int32_t *thrL, int32_t count,
                       uint32_t *bits, hipStream_t s) {
  const int64_t words = (g.n + 31) / 32;
  for (int32_t i0 = 0; i0 < count; i0 += kTinyQueries) {
    const int32_t k = std::min(count - i0, kTinyQueries);
    TinyQueries q = {};
    std::copy(thrU + i0, thrU + i0 + k, q.thrU);
    std::copy(thrL + i0, thrL + i0 + k, q.thrL);
    tiny_kernel<<<k, kTinyBlock, tiny_lds(g), s>>>(g.off, g.cols, g.deg0, (int32_t)g.n, g.nU,
                                                   (int32_t)tiny_items(g), q, bits + i0 * words);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace abc
