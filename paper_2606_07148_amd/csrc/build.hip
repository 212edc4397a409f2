// Device construction of the unified CSR (Sec. III: CSR storage; Sec. IV-A:
// contiguous ids, upper first).  Pairs are keyed (u, v) in two bit fields,
// radix-sorted and deduplicated (E is a set); the sorted keys give the upper
// rows directly.  The sort is stable, so sorting them again by v's field
// alone gives the lower rows.  The sorts are rocPRIM's device radix sort,
// called directly (prim.h) between two buffers; the build is preprocessing
// and is not part of the timed peel.
#include "prim.h"

#include <algorithm>

#include "abcore_internal.h"
#include "wave.h"

namespace abc {

namespace {

// Keys (u << vbits) | v, and *bad set if an endpoint is out of range (its key
// then means nothing and the build ends after the sort).
__global__ void make_keys_kernel(const int32_t *__restrict__ eu, const int32_t *__restrict__ ev,
                                 int64_t m, int32_t nU, int32_t nL, int vbits,
                                 uint64_t *__restrict__ keys, int32_t *bad) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int found = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
    const int32_t u = eu[i], v = ev[i];
    found |= (u < 0 || u >= nU || v < 0 || v >= nL);
    keys[i] = ((uint64_t)(uint32_t)u << vbits) | (uint64_t)(uint32_t)v;
  }
  if (__ballot(found) != 0 && (threadIdx.x & 63) == 0) atomicOr(bad, 1);
}

// Counts one per valid lane into deg[row] where the lanes of a wave hold
// sorted rows (the valid lanes a prefix of the wave): one atomic per run of
// equal rows, so that a hub's entries do not queue on one address.
__device__ __forceinline__ void add_row_runs(int32_t *deg, int32_t row, bool ok) {
  const int lane = (int)(threadIdx.x % kWave);
  const int32_t prev = __shfl_up(row, 1, kWave);
  const bool start = ok && (lane == 0 || prev != row);
  const uint64_t starts = __ballot(start);
  const int nvalid = __popcll(__ballot(ok));
  if (start) {
    const uint64_t above = lane == kWave - 1 ? 0ull : (starts >> (lane + 1)) << (lane + 1);
    const int end = above ? __builtin_ctzll(above) : nvalid;
    atomicAdd(&deg[row], end - lane);
  }
}

// The first key of every run of equal ones, in two passes over the sorted
// keys: the firsts of each tile are counted, and after a prefix sum of the
// counts the second pass writes them and, from the same read, the upper rows.
// Bound by memory (a read, then a read and a write of the keys).  24 M keys:
// 0.64 + 0.06 ms by the library's selection and a pass for the rows, 0.03 +
// 0.09 ms by these.
constexpr int kUniqBlock = 256;
constexpr int kUniqPer = 16;  // keys per lane, 64 consecutive ones to a step
constexpr int64_t kUniqTile = (int64_t)kUniqBlock * kUniqPer;
constexpr int kUniqWaves = kUniqBlock / kWave;

// Loads the wave's kUniqPer steps of a tile; first[q]: the lanes of step q
// that hold the first of a run.
__device__ __forceinline__ void load_firsts(const uint64_t *__restrict__ keys, int64_t m,
                                            int64_t base, uint64_t (&k)[kUniqPer],
                                            uint64_t (&first)[kUniqPer]) {
  const int lane = (int)(threadIdx.x % kWave);
#pragma unroll
  for (int q = 0; q < kUniqPer; ++q) {
    const int64_t i = base + q * kWave + lane;
    k[q] = i < m ? keys[i] : 0;
  }
  uint64_t before = base > 0 && base < m ? keys[base - 1] : 0;  // (wave-uniform)
#pragma unroll
  for (int q = 0; q < kUniqPer; ++q) {
    const int64_t i = base + q * kWave + lane;
    uint64_t p = (uint64_t)__shfl_up((unsigned long long)k[q], 1, kWave);
    if (lane == 0) p = before;
    first[q] = __ballot(i < m && (i == 0 || k[q] != p));
    before = (uint64_t)__shfl((unsigned long long)k[q], kWave - 1, kWave);
  }
}

__global__ __launch_bounds__(kUniqBlock) void count_firsts_kernel(
    const uint64_t *__restrict__ keys, int64_t m, int64_t tiles, int64_t *__restrict__ counts) {
  __shared__ int s_count[kUniqWaves];
  const int wave = threadIdx.x / kWave;
  uint64_t k[kUniqPer], first[kUniqPer];
  load_firsts(keys, m, blockIdx.x * kUniqTile + (int64_t)wave * kUniqPer * kWave, k, first);
  int c = 0;
#pragma unroll
  for (int q = 0; q < kUniqPer; ++q) c += __popcll(first[q]);
  if (threadIdx.x % kWave == 0) s_count[wave] = c;
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < kUniqWaves; ++w) c += s_count[w];
  counts[blockIdx.x] = c;
  if (blockIdx.x == 0) counts[tiles] = 0;  // the sum's last slot is the total
}

// Unique key i = (u, v) -> ukeys[i], cols[i] = nU + v; upper degrees.
__global__ __launch_bounds__(kUniqBlock) void upper_rows_kernel(
    const uint64_t *__restrict__ keys, int64_t m, const int64_t *__restrict__ offs, int32_t nU,
    int vbits, uint64_t *__restrict__ ukeys, int32_t *__restrict__ cols,
    int32_t *__restrict__ deg) {
  __shared__ int s_count[kUniqWaves];
  const int wave = threadIdx.x / kWave, lane = (int)(threadIdx.x % kWave);
  const uint64_t vmask = (1ull << vbits) - 1;
  const int64_t base = blockIdx.x * kUniqTile + (int64_t)wave * kUniqPer * kWave;
  uint64_t k[kUniqPer], first[kUniqPer];
  load_firsts(keys, m, base, k, first);
  int c = 0;
#pragma unroll
  for (int q = 0; q < kUniqPer; ++q) c += __popcll(first[q]);
  if (lane == 0) s_count[wave] = c;
  __syncthreads();
  int64_t at = offs[blockIdx.x];
  for (int w = 0; w < wave; ++w) at += s_count[w];
  const uint64_t lt = ((uint64_t)1 << lane) - 1;
#pragma unroll
  for (int q = 0; q < kUniqPer; ++q) {
    const bool mine = (first[q] >> lane) & 1u;
    const int64_t to = at + __popcll(first[q] & lt);
    if (mine) {
      ukeys[to] = k[q];
      cols[to] = nU + (int32_t)(k[q] & vmask);
    }
    at += __popcll(first[q]);
    // one atomic per run of a row's keys in the step, for its firsts
    const int32_t u = (int32_t)(k[q] >> vbits);
    const int32_t prev = __shfl_up(u, 1, kWave);
    const bool ok = base + q * kWave + lane < m;
    const bool start = ok && (lane == 0 || prev != u);
    const uint64_t starts = __ballot(start);
    if (start) {
      const uint64_t above = lane == kWave - 1 ? 0ull : (starts >> (lane + 1)) << (lane + 1);
      const uint64_t upto = above ? (above & (~above + 1)) - 1 : ~0ull;
      const int n = __popcll(first[q] & upto & ~lt);
      if (n > 0) atomicAdd(&deg[u], n);
    }
  }
}

// Lower side: the keys in (v, u) order -> cols[md + i] = u; lower degrees.
__global__ void lower_rows_kernel(const uint64_t *__restrict__ lkeys, int64_t md, int32_t nU,
                                  int vbits, int32_t *__restrict__ cols,
                                  int32_t *__restrict__ deg) {
  const uint64_t vmask = (1ull << vbits) - 1;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x / kWave) * kWave; b < md;
       b += stride) {
    const int64_t i = b + (int64_t)(threadIdx.x % kWave);
    const bool ok = i < md;
    int32_t v = 0;
    if (ok) {
      const uint64_t k = lkeys[i];
      cols[md + i] = (int32_t)(k >> vbits);
      v = (int32_t)(k & vmask);
    }
    add_row_runs(deg + nU, v, ok);
  }
}

__global__ void widen_kernel(const int32_t *__restrict__ deg, int64_t n,
                             int64_t *__restrict__ out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += stride)
    out[i] = i < n ? (int64_t)deg[i] : 0;
}

// Piece counts of every row (rows longer than kPiece entries are split) and
// split-row flags, each followed by a zero so an exclusive scan yields the
// totals in the last slot.
__global__ void count_pieces_kernel(const int64_t *__restrict__ off, int64_t n,
                                    int64_t *__restrict__ np, int64_t *__restrict__ hv) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x <= n; x += stride) {
    const int64_t d = x < n ? off[x + 1] - off[x] : 0;
    np[x] = d > kPiece ? (d + kPiece - 1) / kPiece : 0;
    hv[x] = d > kPiece ? 1 : 0;
  }
}

__global__ void fill_pieces_kernel(const int64_t *__restrict__ off, int64_t n,
                                   const int64_t *__restrict__ first,
                                   const int64_t *__restrict__ hfirst,
                                   int32_t *__restrict__ piece_row,
                                   int64_t *__restrict__ piece_start,
                                   int32_t *__restrict__ piece_first,
                                   int32_t *__restrict__ heavy_rows) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride) {
    const int64_t d = off[x + 1] - off[x];
    if (d > kPiece) {
      const int64_t f = first[x];
      const int64_t np = (d + kPiece - 1) / kPiece;
      piece_first[x] = (int32_t)f;
      if (heavy_rows != nullptr) heavy_rows[hfirst[x]] = (int32_t)x;
      for (int64_t k = 0; k < np; ++k) {
        piece_row[f + k] = (int32_t)x;
        piece_start[f + k] = off[x] + k * kPiece;
      }
    } else {
      piece_first[x] = -1;
    }
  }
}

// Weight of a row in the pull round: its entries when it is walked as a row
// (a split row is walked by its pieces) plus a fixed cost per row.
constexpr int64_t kRowCost = 4;
__global__ void row_weight_kernel(const int64_t *__restrict__ off, int64_t n,
                                  int64_t *__restrict__ w) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x <= n; x += stride) {
    const int64_t d = x < n ? off[x + 1] - off[x] : 0;
    w[x] = x < n ? (d <= kPiece ? d : 0) + kRowCost : 0;
  }
}

// Bound k of layer p (0 upper, 1 lower): the first row of the layer whose
// exclusive weight prefix reaches k/G of the layer's weight.  The prefix is
// strictly increasing (every row costs at least kRowCost), so bound 0 and
// bound G are the layer's first row and its end.
__global__ void pull_bounds_kernel(const int64_t *__restrict__ pre, int64_t nU, int64_t n, int G,
                                   int32_t *__restrict__ bounds) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= 2 * (G + 1)) return;
  const int p = t / (G + 1), k = t % (G + 1);
  int64_t lo = p == 0 ? 0 : nU, hi = p == 0 ? nU : n;
  const int64_t base = pre[lo];
  const int64_t target = base + (pre[hi] - base) * k / G;
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (pre[mid] >= target)
      hi = mid;
    else
      lo = mid + 1;
  }
  bounds[t] = (int32_t)lo;
}

int bits_for(uint64_t maxkey) {
  int b = 0;
  while (b < 64 && (maxkey >> b) != 0) ++b;
  return std::max(b, 1);
}

}  // namespace

BuildScratch::~BuildScratch() { release(); }

void BuildScratch::release() {
  if (temp) (void)dev_free_async(temp, s);
  if (block) (void)dev_free_async(block, s);
  temp = block = nullptr;
  temp_bytes = 0;
}

hipError_t BuildScratch::reserve(int64_t m, int64_t n) {
  const int64_t words = std::max<int64_t>(m, 2 * (n + 1));
  const hipError_t e = dev_malloc_async(&block, sizeof(uint64_t) * (2 * words + n + 2), s);
  if (e != hipSuccess) return e;
  k0 = static_cast<uint64_t *>(block);
  k1 = k0 + words;
  c = reinterpret_cast<int64_t *>(k1 + words);
  flags = reinterpret_cast<int32_t *>(c + n + 1);
  return hipSuccess;
}

hipError_t BuildScratch::reserve_temp(size_t bytes) {
  if (temp != nullptr && bytes <= temp_bytes) return hipSuccess;
  if (temp) (void)dev_free_async(temp, s);
  temp = nullptr;
  temp_bytes = 0;
  const hipError_t e = dev_malloc_async(&temp, std::max<size_t>(bytes, 16), s);
  if (e == hipSuccess) temp_bytes = std::max<size_t>(bytes, 16);
  return e;
}

// Builds off/cols/deg0 of g (already sized: g.nU, g.nL, g.n set; arrays not
// yet allocated).  Returns a status and sets the error message.
abcore_status build_csr_device(Graph &g, BuildScratch &w, const int32_t *eu, const int32_t *ev,
                               int64_t m, hipStream_t s) {
#define BCHK(x)                                                                     \
  do {                                                                              \
    hipError_t e_ = (x);                                                            \
    if (e_ != hipSuccess) {                                                         \
      set_error("CSR build: %s failed: %s", #x, hipGetErrorString(e_));             \
      return (e_ == hipErrorOutOfMemory) ? ABCORE_ENOMEM : ABCORE_EDEVICE;          \
    }                                                                               \
  } while (0)
  const int grid = std::max(1, std::min(g.cu_count * 8, (int)((m + 255) / 256)));
  size_t need = 0, most = 0;
  int64_t md = 0;
  const int64_t tiles = (m + kUniqTile - 1) / kUniqTile;
  int64_t *offs = nullptr;  // in the temporary storage: the tiles' first unique keys
  const int vbits = bits_for((uint64_t)std::max(g.nL, 1) - 1);
  const int ubits = bits_for((uint64_t)std::max(g.nU, 1) - 1);

  BCHK(dev_malloc(&g.off, sizeof(int64_t) * (g.n + 1)));
  BCHK(dev_malloc(&g.deg0, sizeof(int32_t) * std::max<int64_t>(g.n, 1)));
  BCHK(w.reserve(m, g.n));
  BCHK(hipMemsetAsync(g.deg0, 0, sizeof(int32_t) * std::max<int64_t>(g.n, 1), s));
  if (m > 0) {
    uint64_t *cur = w.k0, *alt = w.k1;
    BCHK(hipMemsetAsync(w.flags, 0, 2 * sizeof(int32_t), s));
    make_keys_kernel<<<grid, 256, 0, s>>>(eu, ev, m, g.nU, g.nL, vbits, cur, w.flags);
    BCHK(hipGetLastError());
    // temporary storage large enough for the sort, then for the tiles' counts
    // and their sums
    BCHK(prim::sort_keys_two(nullptr, need, cur, alt, (size_t)m, 0, ubits + vbits, s));
    most = need;
    BCHK(prim::exclusive_sum(nullptr, need, nullptr, nullptr, (size_t)(tiles + 1), s));
    const size_t sums = 2 * sizeof(int64_t) * (size_t)(tiles + 1);
    BCHK(w.reserve_temp(std::max(most, (sums + 255) / 256 * 256 + need)));
    need = w.temp_bytes;
    BCHK(prim::sort_keys_two(w.temp, need, cur, alt, (size_t)m, 0, ubits + vbits, s));
    int64_t *counts = static_cast<int64_t *>(w.temp);
    offs = counts + tiles + 1;
    count_firsts_kernel<<<(unsigned)tiles, kUniqBlock, 0, s>>>(cur, m, tiles, counts);
    BCHK(hipGetLastError());
    need = w.temp_bytes - (sums + 255) / 256 * 256;
    BCHK(prim::exclusive_sum(static_cast<uint8_t *>(w.temp) + (sums + 255) / 256 * 256, need,
                             counts, offs, (size_t)(tiles + 1), s));
    int32_t bad = 0;
    BCHK(hipMemcpyAsync(&bad, w.flags, sizeof(bad), hipMemcpyDeviceToHost, s));
    BCHK(hipMemcpyAsync(&md, offs + tiles, sizeof(md), hipMemcpyDeviceToHost, s));
    BCHK(hipStreamSynchronize(s));
    if (bad != 0) {
      set_error("abcore_build_csr: edge endpoint out of range");
      return ABCORE_EINVAL;
    }
    w.k0 = alt;  // the unique keys
    w.k1 = cur;
  }
  g.m_csr = md;
  g.m = md;
  BCHK(dev_malloc(&g.cols, sizeof(int32_t) * std::max<int64_t>(2 * md, 1)));
  if (md > 0) {
    const int gridm = std::max(1, std::min(g.cu_count * 8, (int)((md + 255) / 256)));
    upper_rows_kernel<<<(unsigned)tiles, kUniqBlock, 0, s>>>(w.k1, m, offs, g.nU, vbits, w.k0,
                                                             g.cols, g.deg0);
    BCHK(hipGetLastError());
    need = 0;
    BCHK(prim::sort_keys_two(nullptr, need, w.k0, w.k1, (size_t)md, 0, vbits, s));
    BCHK(w.reserve_temp(need));
    need = w.temp_bytes;
    BCHK(prim::sort_keys_two(w.temp, need, w.k0, w.k1, (size_t)md, 0, vbits, s));
    lower_rows_kernel<<<gridm, 256, 0, s>>>(w.k0, md, g.nU, vbits, g.cols, g.deg0);
    BCHK(hipGetLastError());
  }
  {
    const int gridn = std::max(1, std::min(g.cu_count * 8, (int)((g.n + 256) / 256)));
    widen_kernel<<<gridn, 256, 0, s>>>(g.deg0, g.n, w.c);
    BCHK(hipGetLastError());
    need = 0;
    BCHK(prim::exclusive_sum(nullptr, need, w.c, g.off, (size_t)(g.n + 1), s));
    BCHK(w.reserve_temp(need));
    need = w.temp_bytes;
    BCHK(prim::exclusive_sum(w.temp, need, w.c, g.off, (size_t)(g.n + 1), s));
  }
  return ABCORE_OK;
#undef BCHK
}

// Splits rows longer than kPiece entries into pieces (see Graph).
abcore_status build_pieces(Graph &g, BuildScratch &w, hipStream_t s) {
#define PCHK(x)                                                                     \
  do {                                                                              \
    hipError_t e_ = (x);                                                            \
    if (e_ != hipSuccess) {                                                         \
      set_error("piece build: %s failed: %s", #x, hipGetErrorString(e_));           \
      return (e_ == hipErrorOutOfMemory) ? ABCORE_ENOMEM : ABCORE_EDEVICE;          \
    }                                                                               \
  } while (0)
  int64_t *np = reinterpret_cast<int64_t *>(w.k0), *hv = np + (g.n + 1);
  int64_t *first = reinterpret_cast<int64_t *>(w.k1), *hfirst = first + (g.n + 1);
  size_t need = 0;
  int64_t h_tot[4] = {0, 0, 0, 0};
  const int grid = std::max(1, std::min(g.cu_count * 8, (int)((g.n + 256) / 256)));
  count_pieces_kernel<<<grid, 256, 0, s>>>(g.off, g.n, np, hv);
  PCHK(hipGetLastError());
  PCHK(prim::exclusive_sum(nullptr, need, np, first, (size_t)(g.n + 1), s));
  PCHK(w.reserve_temp(need));
  need = w.temp_bytes;
  PCHK(prim::exclusive_sum(w.temp, need, np, first, (size_t)(g.n + 1), s));
  need = w.temp_bytes;
  PCHK(prim::exclusive_sum(w.temp, need, hv, hfirst, (size_t)(g.n + 1), s));
  PCHK(hipMemcpyAsync(&h_tot[0], first + g.n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  PCHK(hipMemcpyAsync(&h_tot[1], first + g.nU, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  PCHK(hipMemcpyAsync(&h_tot[2], hfirst + g.n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  PCHK(hipMemcpyAsync(&h_tot[3], hfirst + g.nU, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  PCHK(hipStreamSynchronize(s));
  g.npieces = h_tot[0];
  g.npieces_upper = h_tot[1];
  g.nheavy = h_tot[2];
  g.nheavy_upper = h_tot[3];
  PCHK(dev_malloc(&g.piece_row, sizeof(int32_t) * std::max<int64_t>(g.npieces, 1)));
  PCHK(dev_malloc(&g.piece_start, sizeof(int64_t) * std::max<int64_t>(g.npieces, 1)));
  PCHK(dev_malloc(&g.piece_first, sizeof(int32_t) * std::max<int64_t>(g.n, 1)));
  PCHK(dev_malloc(&g.heavy_rows, sizeof(int32_t) * std::max<int64_t>(g.nheavy, 1)));
  PCHK(dev_malloc(&g.split_written, sizeof(int32_t) * std::max<int64_t>(g.npieces, 1)));
  fill_pieces_kernel<<<grid, 256, 0, s>>>(g.off, g.n, first, hfirst, g.piece_row, g.piece_start,
                                          g.piece_first, g.heavy_rows);
  PCHK(hipGetLastError());
  // pull round work split (np and hv are free again: weights and prefix)
  g.pull_bounds_grid = g.cu_count;
  PCHK(dev_malloc(&g.pull_bounds, sizeof(int32_t) * 2 * (g.pull_bounds_grid + 1)));
  row_weight_kernel<<<grid, 256, 0, s>>>(g.off, g.n, np);
  PCHK(hipGetLastError());
  need = w.temp_bytes;
  PCHK(prim::exclusive_sum(w.temp, need, np, hv, (size_t)(g.n + 1), s));
  pull_bounds_kernel<<<(2 * (g.pull_bounds_grid + 1) + 255) / 256, 256, 0, s>>>(
      hv, g.nU, g.n, g.pull_bounds_grid, g.pull_bounds);
  PCHK(hipGetLastError());
  return ABCORE_OK;
#undef PCHK
}

namespace {

// Sort keys of the rank order: layer, then decreasing degree, above the id.
// The ids start in order and the sort is stable, so it takes the upper field
// alone (dbits of degree and the layer's bit; top is no smaller than any
// degree).
__global__ void rank_keys_kernel(const int64_t *__restrict__ off, int64_t nU, int64_t n,
                                 int64_t top, int dbits, uint64_t *__restrict__ keys) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride) {
    const uint64_t d = (uint64_t)(off[x + 1] - off[x]);
    keys[x] = ((((uint64_t)(x >= nU) << dbits) | ((uint64_t)top - d)) << 32) | (uint64_t)x;
  }
}

__global__ void rank_scatter_kernel(const uint64_t *__restrict__ sorted, int64_t nU, int64_t n,
                                    const int64_t *__restrict__ off, int32_t *__restrict__ rank,
                                    int32_t *__restrict__ rank_vtx, int64_t *__restrict__ rdeg) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const int64_t x = (int64_t)(uint32_t)sorted[i];
    rank[x] = (int32_t)(i - (i < nU ? 0 : nU));
    rank_vtx[i] = (int32_t)x;
    rdeg[i] = off[x + 1] - off[x];
  }
}

// Entry keys (rank of the upper end << lbits) | rank of the lower end, in
// order of the lower end's rank: the lower rows, taken in rank order.  A
// stable sort by the upper field then gives the upper rows in rank order with
// ascending neighbours, and one more by the lower field the lower rows: two
// sorts of m keys on one layer's bits each, where keying both directions
// with (row, neighbour) sorted 2 m keys on both (at 2e7 edges 2.3 ms of sorts
// against 0.9).  A wave takes 64 rows of at most kPiece entries, or 64
// pieces of longer rows, entry-balanced; bound by the random rank lookups.
__device__ __forceinline__ void emit_entry_keys(const int32_t *__restrict__ cols,
                                                const int32_t *__restrict__ rank, int64_t s,
                                                int d, int64_t shift, int32_t r, int lbits,
                                                uint64_t *__restrict__ keys) {
  constexpr int kU = 4;  // entries in flight per lane
  const int incl = wave_incl_scan(d);
  const int total = __shfl(incl, kWave - 1, kWave);
  const int64_t from = s - (incl - d);
  for (int base = 0; base < total; base += kU * kWave) {
    int32_t w[kU], row[kU];
    int64_t to[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int kk = min(base + u * kWave + lane_id(), total - 1);
      int j = 0;
#pragma unroll
      for (int step = 32; step > 0; step >>= 1)
        if (__shfl(incl, j + step - 1, kWave) <= kk) j += step;
      const int64_t pos = __shfl(from, j, kWave) + kk;
      to[u] = pos + __shfl(shift, j, kWave);
      row[u] = __shfl(r, j, kWave);
      w[u] = cols[pos];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) w[u] = rank[w[u]];
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (base + u * kWave + lane_id() < total)
        keys[to[u]] = ((uint64_t)(uint32_t)w[u] << lbits) | (uint64_t)(uint32_t)row[u];
  }
}

__global__ __launch_bounds__(kBlock) void entry_keys_kernel(
    const int64_t *__restrict__ off, const int32_t *__restrict__ cols,
    const int32_t *__restrict__ rank, const int32_t *__restrict__ rank_vtx,
    const int64_t *__restrict__ roff, const int32_t *__restrict__ rp_row,
    const int64_t *__restrict__ rp_start, int64_t nU, int64_t n, int64_t m, int64_t p0, int64_t p1,
    int lbits, uint64_t *__restrict__ keys) {
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + wave_in_block();
  const int64_t nw = (int64_t)gridDim.x * kWavesPerBlock;
  // (the lower rows' entries are the last m of the rank rows)
  for (int64_t b = p0 + gw * kWave; b < p1; b += nw * kWave) {
    const int64_t p = b + lane_id();
    int64_t s = 0, shift = 0;
    int32_t row = 0;
    int d = 0;
    if (p < p1) {
      row = rp_row[p];
      const int64_t t = rp_start[p], rs = roff[row];
      s = off[rank_vtx[row]] + (t - rs);
      shift = t - m - s;
      d = (int)(min(t + kPiece, roff[row + 1]) - t);
    }
    emit_entry_keys(cols, rank, s, d, shift, row - (int32_t)nU, lbits, keys);
  }
  for (int64_t b = nU + gw * kWave; b < n; b += nw * kWave) {
    const int64_t row = b + lane_id();
    int64_t s = 0, shift = 0;
    int d = 0;
    if (row < n) {
      const int64_t t = roff[row], len = roff[row + 1] - t;
      s = off[rank_vtx[row]];
      shift = t - m - s;
      d = len <= kPiece ? (int)len : 0;
    }
    emit_entry_keys(cols, rank, s, d, shift, (int32_t)(row - nU), lbits, keys);
  }
}

// The rank rows' entries: global ranks (a lower neighbour of an upper row is
// its layer rank past nU, so that the rank rows form a CSR graph of their
// own).
__global__ void entry_unkey_kernel(const uint64_t *__restrict__ keys, int64_t m, int shift,
                                   uint64_t mask, int32_t base, int32_t *__restrict__ out) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride)
    out[i] = (int32_t)((keys[i] >> shift) & mask) + base;
}

// Degree counts by threshold, from the rank order (degrees decrease along a
// layer's ranks): at the last rank of each run of equal degrees d, the
// layer's vertices of degree >= d and their entries.
__global__ void rank_table_kernel(const int64_t *__restrict__ roff, int64_t lo, int64_t hi,
                                  int64_t *__restrict__ ge_cnt, int64_t *__restrict__ ge_ent) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t r = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < hi; r += stride) {
    const int64_t d = roff[r + 1] - roff[r];
    const int64_t dn = r + 1 < hi ? roff[r + 2] - roff[r + 1] : -1;
    if (d != dn) {
      ge_cnt[d] = r + 1 - lo;
      ge_ent[d] = roff[r + 1] - roff[lo];
    }
  }
}

}  // namespace

abcore_status build_ranks(Graph &g, BuildScratch &w, hipStream_t s) {
  const int64_t m = g.m_csr, ent = 2 * m;
  if (g.n == 0) return ABCORE_OK;
  // row positions are kept in 31 bits elsewhere; larger graphs keep the
  // bitmap pull
  if (ent >= 0x7FFFFFFFLL) return ABCORE_OK;
  uint64_t *k0 = w.k0, *k1 = w.k1;
  bool ok = true;
  const int grid = std::max(1, std::min(g.cu_count * 8, (int)((g.n + 255) / 256)));
  const int64_t top = std::max<int64_t>(std::max<int64_t>(g.nU, g.nL), 1);  // >= any degree
  const int dbits = bits_for((uint64_t)top);
  const int ubits = bits_for((uint64_t)std::max(g.nU, 1) - 1);
  const int lbits = bits_for((uint64_t)std::max(g.nL, 1) - 1);
  const int xbits = bits_for((uint64_t)std::max<int64_t>(g.n, 1) - 1);
  auto fail = [&](hipError_t e) {
    if (e != hipSuccess) ok = false;
    return e != hipSuccess;
  };
  auto sort_bits = [&](int64_t count, int begin, int end) {
    size_t need = 0;
    hipError_t e = prim::sort_keys_two(nullptr, need, k0, k1, (size_t)count, begin, end, s);
    if (e == hipSuccess) e = w.reserve_temp(need);
    need = w.temp_bytes;
    return e == hipSuccess
               ? prim::sort_keys_two(w.temp, need, k0, k1, (size_t)count, begin, end, s)
               : e;
  };
  auto sum = [&](const int64_t *in, int64_t *out) {
    size_t need = 0;
    hipError_t e = prim::exclusive_sum(nullptr, need, in, out, (size_t)(g.n + 1), s);
    if (e == hipSuccess) e = w.reserve_temp(need);
    need = w.temp_bytes;
    return e == hipSuccess ? prim::exclusive_sum(w.temp, need, in, out, (size_t)(g.n + 1), s) : e;
  };
  do {
    if (fail(dev_malloc(&g.rank, sizeof(int32_t) * g.n))) break;
    if (fail(dev_malloc(&g.rank_vtx, sizeof(int32_t) * g.n))) break;
    if (fail(dev_malloc(&g.roff, sizeof(int64_t) * (g.n + 1)))) break;
    if (fail(dev_malloc(&g.rcols, sizeof(int32_t) * std::max<int64_t>(ent, 1)))) break;
    g.rdeg_mask = (uint32_t)((1ull << xbits) - 1);
    if (fail(dev_malloc(&g.rdeg, sizeof(int32_t) * ((size_t)g.rdeg_mask + 1)))) break;
    if (fail(dev_malloc(&g.rp_row, sizeof(int32_t) * std::max<int64_t>(g.npieces, 1)))) break;
    if (fail(dev_malloc(&g.rp_start, sizeof(int64_t) * std::max<int64_t>(g.npieces, 1)))) break;
    if (fail(dev_malloc(&g.rp_first, sizeof(int32_t) * g.n))) break;
    // ranks, both layers at once; their degrees place the rank rows
    rank_keys_kernel<<<grid, 256, 0, s>>>(g.off, g.nU, g.n, top, dbits, k0);
    if (fail(hipGetLastError())) break;
    if (fail(sort_bits(g.n, 32, 32 + dbits + 1))) break;
    rank_scatter_kernel<<<grid, 256, 0, s>>>(k0, g.nU, g.n, g.off, g.rank, g.rank_vtx, w.c);
    if (fail(hipGetLastError())) break;
    if (fail(hipMemsetAsync(w.c + g.n, 0, sizeof(int64_t), s))) break;
    if (fail(sum(w.c, g.roff))) break;
    // the rank rows' pieces (the same lengths as the vertex rows', in rank
    // order; the key buffers serve as the counts and their scans)
    {
      int64_t *np = reinterpret_cast<int64_t *>(k0), *hv = np + (g.n + 1);
      int64_t *first = reinterpret_cast<int64_t *>(k1);
      count_pieces_kernel<<<grid, 256, 0, s>>>(g.roff, g.n, np, hv);
      if (fail(hipGetLastError())) break;
      if (fail(sum(np, first))) break;
      fill_pieces_kernel<<<grid, 256, 0, s>>>(g.roff, g.n, first, nullptr, g.rp_row, g.rp_start,
                                              g.rp_first, nullptr);
      if (fail(hipGetLastError())) break;
    }
    if (m > 0) {
      entry_keys_kernel<<<wide_grid(g), kBlock, 0, s>>>(
          g.off, g.cols, g.rank, g.rank_vtx, g.roff, g.rp_row, g.rp_start, g.nU, g.n, m,
          g.npieces_upper, g.npieces, lbits, k0);
      if (fail(hipGetLastError())) break;
      if (fail(sort_bits(m, lbits, lbits + ubits))) break;
      const int gridm = std::max(1, std::min(g.cu_count * 8, (int)((m + 255) / 256)));
      entry_unkey_kernel<<<gridm, 256, 0, s>>>(k0, m, 0, (1ull << lbits) - 1, g.nU, g.rcols);
      if (fail(hipGetLastError())) break;
      if (fail(sort_bits(m, 0, lbits))) break;
      entry_unkey_kernel<<<gridm, 256, 0, s>>>(k0, m, lbits, (1ull << ubits) - 1, 0, g.rcols + m);
      if (fail(hipGetLastError())) break;
    }
    // per layer and threshold t: the vertices of degree >= t (ranks [0, K))
    // and their entries, kept on the host
    for (int layer = 0; layer < 2 && ok; ++layer) {
      const int64_t lo = layer == 0 ? 0 : g.nU, hi = layer == 0 ? g.nU : g.n;
      g.rk_cnt[layer].assign(1, 0);
      g.rk_ent[layer].assign(1, 0);
      if (hi <= lo) continue;
      int64_t r01[2] = {0, 0};
      if (fail(hipMemcpyAsync(r01, g.roff + lo, sizeof(int64_t) * 2, hipMemcpyDeviceToHost, s)))
        break;
      if (fail(hipStreamSynchronize(s))) break;
      const int64_t maxdeg = r01[1] - r01[0];
      // (k0 and k1 are free again and hold at least n + 1 values each)
      int64_t *gc = reinterpret_cast<int64_t *>(k0), *ge = reinterpret_cast<int64_t *>(k1);
      if (maxdeg + 1 > g.n + 1) {
        ok = false;
        break;
      }
      if (fail(hipMemsetAsync(gc, 0xFF, sizeof(int64_t) * (maxdeg + 1), s))) break;
      rank_table_kernel<<<grid, 256, 0, s>>>(g.roff, lo, hi, gc, ge);
      if (fail(hipGetLastError())) break;
      std::vector<int64_t> hc(maxdeg + 1), he(maxdeg + 1);
      if (fail(hipMemcpyAsync(hc.data(), gc, sizeof(int64_t) * (maxdeg + 1),
                              hipMemcpyDeviceToHost, s)))
        break;
      if (fail(hipMemcpyAsync(he.data(), ge, sizeof(int64_t) * (maxdeg + 1),
                              hipMemcpyDeviceToHost, s)))
        break;
      if (fail(hipStreamSynchronize(s))) break;
      // a degree no vertex has takes the counts of the next larger one
      std::vector<int64_t> &kc = g.rk_cnt[layer], &ke = g.rk_ent[layer];
      kc.assign(maxdeg + 2, 0);
      ke.assign(maxdeg + 2, 0);
      for (int64_t t = maxdeg; t >= 0; --t) {
        kc[t] = hc[t] >= 0 ? hc[t] : kc[t + 1];
        ke[t] = hc[t] >= 0 ? he[t] : ke[t + 1];
      }
    }
    if (!ok) break;
    if (fail(hipStreamSynchronize(s))) break;
  } while (0);
  w.k0 = k0;
  w.k1 = k1;
  if (!ok) {
    (void)hipGetLastError();
    if (g.rank) (void)dev_free(g.rank);
    if (g.rank_vtx) (void)dev_free(g.rank_vtx);
    if (g.roff) (void)dev_free(g.roff);
    if (g.rcols) (void)dev_free(g.rcols);
    if (g.rdeg) (void)dev_free(g.rdeg);
    g.rdeg = nullptr;
    g.rdeg_mask = 0;
    if (g.rp_row) (void)dev_free(g.rp_row);
    if (g.rp_start) (void)dev_free(g.rp_start);
    if (g.rp_first) (void)dev_free(g.rp_first);
    g.rank = nullptr;
    g.rank_vtx = nullptr;
    g.roff = nullptr;
    g.rcols = nullptr;
    g.rp_row = nullptr;
    g.rp_start = nullptr;
    g.rp_first = nullptr;
    for (int layer = 0; layer < 2; ++layer) {
      g.rk_cnt[layer].clear();
      g.rk_ent[layer].clear();
    }
  }
  return ABCORE_OK;
}

}  // namespace abc
