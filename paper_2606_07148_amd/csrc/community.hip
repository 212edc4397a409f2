// Vertex sets around a query (Remark of Sec. V): after a peel scoped to the
// component(s) of one or two vertices -- GFQ's Algorithm 1 on the affected
// component, or the same for a static query vertex -- the result is either
// every survivor of that scope (the vertices the scoped peel leaves) or only
// those connected to the query vertices through survivors (the connected
// part of the (alpha,beta)-core that holds them, by a union-find over the
// core's induced subgraph).
#include "abcore_internal.h"
#include "wave.h"

namespace abc {

// Bit x of `bits`: x lies in the component of vx or of vy (labels read from
// comp, which the scoped scan used) and its final working degree reached its
// threshold.  Every word is written; *count (nullable) gains the bits set.
// connected: a component counts only if its vx or vy is such a vertex itself,
// so that the search for the parts around vertices outside the core passes
// over empty words.
__global__ __launch_bounds__(kBlock) void pack_scope_kernel(const int32_t *__restrict__ deg,
                                                            const int32_t *__restrict__ comp,
                                                            int32_t vx, int32_t vy, int64_t n,
                                                            int32_t nU, int32_t thrU,
                                                            int32_t thrL,
                                                            uint32_t *__restrict__ bits,
                                                            int64_t nwords, bool connected,
                                                            unsigned long long *count) {
  auto label = [&](int32_t v) {
    const int32_t c = comp[v], d = ld_agent(&deg[v]);
    return connected && d < (v < nU ? thrU : thrL) ? -1 : c;  // (no vertex has label -1)
  };
  const int32_t c1 = label(vx), c2 = label(vy);
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  unsigned long long total = 0;
  for (int64_t base = ((int64_t)blockIdx.x * kWavesPerBlock + wave_in_block()) * kWave;
       base < nwords * 32; base += stride) {
    const int64_t x = base + lane_id();
    bool p = false;
    if (x < n) {
      const int32_t c = comp[x];
      p = (c == c1 || c == c2) && ld_agent(&deg[x]) >= (x < nU ? thrU : thrL);
    }
    const uint64_t mask = __ballot(p);
    const int64_t w0 = base / 32;
    if (lane_id() == 0) {
      bits[w0] = (uint32_t)mask;
      total += __popcll(mask);
    }
    if (lane_id() == 1 && w0 + 1 < nwords) bits[w0 + 1] = (uint32_t)(mask >> 32);
  }
  if (count == nullptr) return;
  __shared__ unsigned long long s;
  if (threadIdx.x == 0) s = 0;
  __syncthreads();
  if (total != 0) atomicAdd(&s, total);
  __syncthreads();
  if (threadIdx.x == 0 && s != 0) atomicAdd(count, s);
}

__global__ __launch_bounds__(kBlock) void popcount_kernel(const uint32_t *__restrict__ w,
                                                          int64_t nwords,
                                                          unsigned long long *out) {
  __shared__ unsigned long long s;
  if (threadIdx.x == 0) s = 0;
  __syncthreads();
  unsigned long long c = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nwords; i += stride)
    c += (unsigned long long)__popc(w[i]);
  atomicAdd(&s, c);
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(out, s);
}

// The largest degree over ids [lo, hi) into *out (which must start at 0).
__global__ __launch_bounds__(kBlock) void max_deg_kernel(const int32_t *__restrict__ deg0,
                                                         int64_t lo, int64_t hi, int32_t *out) {
  __shared__ int32_t s;
  if (threadIdx.x == 0) s = 0;
  __syncthreads();
  int32_t m = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < hi; i += stride)
    m = max(m, deg0[i]);
  atomicMax(&s, m);
  __syncthreads();
  if (threadIdx.x == 0) atomicMax(out, s);
}

static int grid_for(const Graph &g, int64_t items, int per_block) {
  const int64_t b = (items + per_block - 1) / per_block;
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, std::min(g.cu_count * 8, kMaxBlocks)));
}

// The vertex set after a peel scoped to the components of vx and vy (their
// labels in g.comp): every survivor of the scope, or with `connected` the
// survivors reachable from vx or vy through survivors.  Writes every word of
// d_bits; *count (nullable) receives the set's size.  Synchronous.
abcore_status scoped_set(Graph &g, int32_t vx, int32_t vy, int32_t thrU, int32_t thrL,
                         bool connected, uint32_t *d_bits, int64_t *count, hipStream_t s) {
  const int64_t nwords = (g.n + 31) / 32;
  if (g.aux == nullptr) {
    if (dev_malloc(&g.aux, sizeof(int64_t) * 4) != hipSuccess) {
      g.aux = nullptr;
      set_error("community: allocation of counters failed");
      return ABCORE_ENOMEM;
    }
  }
  unsigned long long h = 0;
  unsigned long long *dc = reinterpret_cast<unsigned long long *>(g.aux) + 2;
  uint32_t *member = connected ? g.row_bits : d_bits;
  if (hipMemsetAsync(dc, 0, sizeof(unsigned long long), s) != hipSuccess) goto fail;
  pack_scope_kernel<<<grid_for(g, nwords * 32, kBlock), kBlock, 0, s>>>(
      g.deg, g.comp, vx, vy, g.n, g.nU, thrU, thrL, member, nwords, connected,
      connected ? nullptr : dc);
  if (hipGetLastError() != hipSuccess) goto fail;
  if (connected && launch_reached(g, member, vx, vy, d_bits, dc, s) != hipSuccess) goto fail;
  if (count != nullptr &&
      hipMemcpyAsync(&h, dc, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess)
    goto fail;
  if (hipStreamSynchronize(s) != hipSuccess) goto fail;
  if (count != nullptr) *count = (int64_t)h;
  return ABCORE_OK;
fail:
  set_error("community: a device call failed");
  return ABCORE_EDEVICE;
}

abcore_status max_degree(Graph &g, int64_t lo, int64_t hi, int32_t *out, hipStream_t s) {
  if (g.aux == nullptr && dev_malloc(&g.aux, sizeof(int64_t) * 4) != hipSuccess) {
    g.aux = nullptr;
    set_error("offsets: allocation of counters failed");
    return ABCORE_ENOMEM;
  }
  int32_t *d = reinterpret_cast<int32_t *>(g.aux);
  int32_t h = 0;
  if (hipMemsetAsync(d, 0, sizeof(int32_t), s) != hipSuccess) goto fail;
  if (hi > lo) {
    max_deg_kernel<<<grid_for(g, hi - lo, kBlock), kBlock, 0, s>>>(g.deg0, lo, hi, d);
    if (hipGetLastError() != hipSuccess) goto fail;
  }
  if (hipMemcpyAsync(&h, d, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    goto fail;
  *out = h;
  return ABCORE_OK;
fail:
  set_error("offsets: a device call failed");
  return ABCORE_EDEVICE;
}

abcore_status count_bits(Graph &g, const uint32_t *bits, int64_t *out, hipStream_t s) {
  if (g.aux == nullptr && dev_malloc(&g.aux, sizeof(int64_t) * 4) != hipSuccess) {
    g.aux = nullptr;
    set_error("allocation of counters failed");
    return ABCORE_ENOMEM;
  }
  const int64_t nwords = (g.n + 31) / 32;
  unsigned long long h = 0;
  unsigned long long *dc = reinterpret_cast<unsigned long long *>(g.aux) + 2;
  if (hipMemsetAsync(dc, 0, sizeof(unsigned long long), s) != hipSuccess) goto fail;
  if (nwords > 0) {
    popcount_kernel<<<grid_for(g, nwords, kBlock), kBlock, 0, s>>>(bits, nwords, dc);
    if (hipGetLastError() != hipSuccess) goto fail;
  }
  if (hipMemcpyAsync(&h, dc, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    goto fail;
  *out = (int64_t)h;
  return ABCORE_OK;
fail:
  set_error("counting bits: a device call failed");
  return ABCORE_EDEVICE;
}

}  // namespace abc
