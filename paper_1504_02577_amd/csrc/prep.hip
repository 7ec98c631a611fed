// Graph preparation (Eq. 3's transition step): CSR validation, per-row
// weight sums W_v, the start set {v : W_v > 0}, per-row inclusive weight
// prefixes and guide records, plus the device-wide exclusive scan used here
// and by the index.
#include "common.h"
#include "kernels.h"

namespace panther {

namespace {

constexpr int kBlock = 256;

__global__ void __launch_bounds__(kBlock)
k_validate(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col, int32_t n,
           int64_t m, uint32_t* err) {
  const int64_t gid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t gsz = (int64_t)gridDim.x * kBlock;
  uint32_t e = 0;
  for (int64_t v = gid; v < n; v += gsz)
    if (row_ptr[v + 1] < row_ptr[v]) e |= 1u;
  for (int64_t i = gid; i < m; i += gsz) {
    const int32_t c = col[i];
    if (c < 0 || c >= n) e |= 2u;
  }
  if (e) atomicOr(err, e);
}

// Symmetry check of an undirected CSR (Sec. 2, Definition 1: E holds
// unordered pairs, so the entry v->u of weight w is stored in both rows).
// Pass 1 marks the rows whose columns ascend; pass 2 takes one wavefront
// per row and, for every entry (v, u, w), compares how many entries of row v
// read (u, w) with how many of row u read (v, w) -- multi-edges must match
// in number.  Ascending rows are searched by bisection, others scanned.
__global__ void __launch_bounds__(kBlock)
k_rows_sorted(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col, int32_t n,
              uint8_t* __restrict__ sorted) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t wave = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
  const int64_t nwaves = (int64_t)gridDim.x * (kBlock / kWave);
  for (int64_t v = wave; v < n; v += nwaves) {
    const int32_t a = row_ptr[v], b = row_ptr[v + 1];
    bool ok = true;
    for (int32_t e = a + 1 + lane; e < b; e += kWave) ok = ok && col[e - 1] <= col[e];
    const bool all = __ballot(!ok) == 0ull;
    if (lane == 0) sorted[v] = all ? 1 : 0;
  }
}

// Entries of row r equal to (t, wt).
__device__ __forceinline__ uint32_t row_matches(const int32_t* __restrict__ row_ptr,
                                                const int32_t* __restrict__ col,
                                                const uint32_t* __restrict__ w,
                                                const uint8_t* __restrict__ sorted, int32_t r,
                                                int32_t t, uint32_t wt) {
  int32_t lo = row_ptr[r];
  const int32_t hi = row_ptr[r + 1];
  uint32_t c = 0;
  if (sorted[r]) {
    int32_t h = hi;
    while (lo < h) {  // first entry with col >= t
      const int32_t mid = lo + ((h - lo) >> 1);
      if (col[mid] < t)
        lo = mid + 1;
      else
        h = mid;
    }
    for (int32_t e = lo; e < hi && col[e] == t; ++e) c += w[e] == wt ? 1u : 0u;
  } else {
    for (int32_t e = lo; e < hi; ++e) c += (col[e] == t && w[e] == wt) ? 1u : 0u;
  }
  return c;
}

__global__ void __launch_bounds__(kBlock)
k_check_symmetric(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                  const uint32_t* __restrict__ w, const uint8_t* __restrict__ sorted, int32_t n,
                  uint32_t* err) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t wave = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
  const int64_t nwaves = (int64_t)gridDim.x * (kBlock / kWave);
  bool bad = false;
  for (int64_t v = wave; v < n; v += nwaves) {
    const int32_t a = row_ptr[v], b = row_ptr[v + 1];
    for (int32_t e = a + lane; e < b; e += kWave) {
      const int32_t u = col[e];
      const uint32_t wt = w[e];
      if (u == (int32_t)v) continue;  // a self-loop is its own reverse
      if (row_matches(row_ptr, col, w, sorted, (int32_t)v, u, wt) !=
          row_matches(row_ptr, col, w, sorted, u, (int32_t)v, wt))
        bad = true;
    }
  }
  if (__ballot(bad) != 0ull && lane == 0) atomicOr(err, 4u);
}

// ---- per-row sums, prefixes and guide records, all from one device-wide
// scan of the weights: sum[e] = the weights of the entries before e (below
// 2^63: fewer than 2^31 entries of 32 bits), so W_v and every row prefix are
// differences of two of its values and no kernel depends on row lengths.
// (One thread per short row and one wave per long row took 23.0 ms of an
// R-MAT 22 load, 128 million entries, most of it waiting for the longest
// rows; these kernels and the scan take 5.6 ms, of which the records, 8.2 GB
// written, 4.4.)

// Entries per work-group of the per-entry kernels; row_of finds an entry's
// row between those of the first entries of its tile and the next.
constexpr int kEdgePer = 16;
constexpr int kEdgeTile = kBlock * kEdgePer;

__global__ void __launch_bounds__(kBlock)
k_rows(const int32_t* __restrict__ row_ptr, const uint64_t* __restrict__ sum, int32_t n,
       int start_all, VRec* __restrict__ vrec, uint64_t* __restrict__ base,
       uint32_t* __restrict__ flags, int32_t* __restrict__ tile_row, unsigned long long* max_w) {
  const int32_t v = blockIdx.x * kBlock + threadIdx.x;
  uint64_t W = 0;
  if (v < n) {
    const int32_t a = row_ptr[v], b = row_ptr[v + 1];
    const uint64_t s = sum[a];
    W = sum[b] - s;
    vrec[v] = VRec{a, b - a, (uint32_t)W, (uint32_t)(W >> 32)};
    base[v] = s;
    flags[v] = (start_all || W) ? 1u : 0u;
    // the tiles whose first entry is in this row
    for (int64_t t = ((int64_t)a + kEdgeTile - 1) / kEdgeTile; t * kEdgeTile < b; ++t)
      tile_row[t] = v;
  }
  W = wave_max(W);
  // Only a wave above the maximum so far writes it: with all 65,536 waves of
  // 4 M rows writing that one address the kernel took 0.75 ms instead of 0.13.
  if ((threadIdx.x & (kWave - 1)) == 0 &&
      W > __hip_atomic_load(max_w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(max_w, (unsigned long long)W);
}

// The row holding entry e: the last v in [lo, hi] with row_ptr[v] <= e (its
// row is not empty, since row_ptr[v + 1] > e).
__device__ __forceinline__ int32_t row_of(const int32_t* __restrict__ row_ptr, int32_t lo,
                                          int32_t hi, int32_t e) {
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo + 1) >> 1);
    if (row_ptr[mid] <= e)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// The rows of one tile's entries: their starts are kept in LDS when they are
// few (every tile but those among long runs of empty rows), so that the
// bisection of each entry (eight steps at 30 entries a row) stays there
// (k_edges32 at 128 M entries: 1.14 -> 0.49 ms).
constexpr int kRowCache = 2048;
struct TileRows {
  const int32_t* row_ptr;
  int32_t* cache;  // [kRowCache] LDS
  int32_t lo, hi;
  bool cached;
  __device__ __forceinline__ void load(const int32_t* rp, const int32_t* tile_row, int32_t n,
                                       int32_t* lds) {
    row_ptr = rp;
    cache = lds;
    lo = tile_row[blockIdx.x];
    hi = blockIdx.x + 1 < gridDim.x ? tile_row[blockIdx.x + 1] : n - 1;
    cached = hi - lo < kRowCache;
    if (cached)
      for (int32_t i = threadIdx.x; i <= hi - lo; i += kBlock) cache[i] = rp[lo + i];
    __syncthreads();
  }
  __device__ __forceinline__ int32_t of(int32_t e) const {
    return cached ? lo + row_of(cache, 0, hi - lo, e) : row_of(row_ptr, lo, hi, e);
  }
};

// edge[e] = {inclusive weight prefix, column}: one 8-byte load gives both.
__global__ void __launch_bounds__(kBlock)
k_edges32(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ tile_row,
          const uint64_t* __restrict__ sum, const uint64_t* __restrict__ base,
          const int32_t* __restrict__ col, int32_t n, int64_t m, uint2* __restrict__ edge) {
  __shared__ int32_t s_rows[kRowCache];
  TileRows rows;
  rows.load(row_ptr, tile_row, n, s_rows);
  const int64_t e0 = (int64_t)blockIdx.x * kEdgeTile + threadIdx.x;
#pragma unroll 4
  for (int i = 0; i < kEdgePer; ++i) {
    const int64_t e = e0 + i * kBlock;
    if (e >= m) break;
    const int32_t v = rows.of((int32_t)e);
    edge[e] = make_uint2((uint32_t)(sum[e + 1] - base[v]), (uint32_t)col[e]);
  }
}

// 64-bit prefixes; in place when pfx == sum + 1 (each entry's own slot).
__global__ void __launch_bounds__(kBlock)
k_prefix64(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ tile_row,
           const uint64_t* sum, const uint64_t* __restrict__ base, int32_t n, int64_t m,
           uint64_t* pfx) {
  __shared__ int32_t s_rows[kRowCache];
  TileRows rows;
  rows.load(row_ptr, tile_row, n, s_rows);
  const int64_t e0 = (int64_t)blockIdx.x * kEdgeTile + threadIdx.x;
#pragma unroll 4
  for (int i = 0; i < kEdgePer; ++i) {
    const int64_t e = e0 + i * kBlock;
    if (e >= m) break;
    const int32_t v = rows.of((int32_t)e);
    pfx[e] = sum[e + 1] - base[v];
  }
}

// Start set: vertex ids and, for the walk's first step, {vertex, row start,
// degree, W} records (one 16-byte load instead of two lines).
__global__ void __launch_bounds__(kBlock)
k_start_scatter(const uint32_t* __restrict__ flags, const uint64_t* __restrict__ pos,
                const VRec* __restrict__ vrec, int32_t n, int32_t* __restrict__ vstart,
                int4* __restrict__ rec) {
  const int32_t v = blockIdx.x * kBlock + threadIdx.x;
  if (v >= n || !flags[v]) return;
  const uint64_t i = pos[v];
  vstart[i] = v;
  if (rec) {
    const VRec r = vrec[v];
    rec[i] = make_int4(v, r.start, r.deg, (int32_t)r.w_lo);
  }
}

// Guide entry b of a row of degree d: the draws r with floor(r d / 2^64) = b
// are r in [ceil(b 2^64 / d), ceil((b+1) 2^64 / d)); the smallest of them
// gives the smallest u = floor(r W / 2^64), and the first edge with prefix
// > that u is where the selection for any draw of the bucket can start.
// ceil(b 2^64 / d) = b Q + ceil(b Rm / d) with Q = floor(2^64 / d) and
// Rm = 2^64 mod d, all in 64-bit integers.
template <typename PrefixFn>
__device__ __forceinline__ int32_t guide_entry(PrefixFn pfx, int32_t start, int32_t deg,
                                               uint64_t W, uint64_t b) {
  const uint64_t d = (uint64_t)deg;
  uint64_t Q = ~0ull / d;
  uint64_t Rm = ~0ull - Q * d + 1ull;
  if (Rm == d) {
    Q += 1ull;
    Rm = 0ull;
  }
  const uint64_t rmin = b * Q + (b * Rm + d - 1ull) / d;
  const uint64_t u = __umul64hi(rmin, W);
  int32_t lo = start, hi = start + deg - 1;
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    if ((uint64_t)pfx(mid) > u)
      hi = mid;
    else
      lo = mid + 1;
  }
  return lo;
}

// Fat guide record of bucket b (four 16-byte chunks): the inclusive prefixes
// of the first three candidate edges from the guide entry e0 onward and e0
// itself, then each candidate's {column, target's row start, target's
// degree, target's W}.  Candidates past the row end repeat the last edge,
// whose prefix W_v exceeds every draw, so they are never preferred.
// One thread per bucket: neighbouring buckets of a row bisect and gather
// nearly the same entries, so those loads meet in L1, and the lanes of a
// quad exchange chunks so that a record leaves as one 64-byte store.
__global__ void __launch_bounds__(kBlock)
k_guide32(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ tile_row,
          const VRec* __restrict__ vrec, const uint2* __restrict__ edge, int32_t n, int64_t m,
          uint4* __restrict__ fat) {
  __shared__ int32_t s_rows[kRowCache];
  TileRows rows;
  rows.load(row_ptr, tile_row, n, s_rows);
  const int64_t t0 = (int64_t)blockIdx.x * kEdgeTile + threadIdx.x;
  const int p = threadIdx.x & 3;
#pragma unroll 1
  for (int i = 0; i < kEdgePer; ++i) {
    const int64_t at = t0 + i * kBlock;
    // lanes past the last bucket repeat it: their quad needs every lane
    const int32_t e = (int32_t)(at < m ? at : m - 1);
    const int32_t v = rows.of(e);
    const VRec r = vrec[v];
    uint4 g[4] = {};
    if (r.w_lo) {  // a weightless row has no record
      const int32_t last = r.start + r.deg - 1;
      const int32_t c0 = guide_entry([&](int32_t x) { return edge[x].x; }, r.start, r.deg,
                                     (uint64_t)r.w_lo, (uint64_t)(e - r.start));
      uint2 y[3];
      VRec t[3];
#pragma unroll
      for (int j = 0; j < 3; ++j) y[j] = edge[c0 + j < last ? c0 + j : last];
#pragma unroll
      for (int j = 0; j < 3; ++j) t[j] = vrec[y[j].y];
      g[0] = make_uint4(y[0].x, y[1].x, y[2].x, (uint32_t)c0);
#pragma unroll
      for (int j = 0; j < 3; ++j)
        g[j + 1] = make_uint4(y[j].y, (uint32_t)t[j].start, (uint32_t)t[j].deg, t[j].w_lo);
    }
    quad_exchange(g);
    // chunk p of the records of the quad's four buckets
    const int64_t q = at - p;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (q + j < m) fat[4 * (q + j) + p] = g[j];
  }
}

// The same for 64-bit prefixes: two candidates, [pfx0 pfx1] [col st dg e0]
// [col st dg -] [W0 W1].
__global__ void __launch_bounds__(kBlock)
k_guide64(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ tile_row,
          const VRec* __restrict__ vrec, const uint64_t* __restrict__ pfx,
          const int32_t* __restrict__ col, int32_t n, int64_t m, uint4* __restrict__ fat) {
  __shared__ int32_t s_rows[kRowCache];
  TileRows rows;
  rows.load(row_ptr, tile_row, n, s_rows);
  const int64_t t0 = (int64_t)blockIdx.x * kEdgeTile + threadIdx.x;
  const int p = threadIdx.x & 3;
#pragma unroll 1
  for (int i = 0; i < kEdgePer; ++i) {
    const int64_t at = t0 + i * kBlock;
    const int32_t e = (int32_t)(at < m ? at : m - 1);
    const int32_t v = rows.of(e);
    const VRec r = vrec[v];
    uint4 g[4] = {};
    if (r.w_lo | r.w_hi) {
      const int32_t last = r.start + r.deg - 1;
      const int32_t c0 = guide_entry([&](int32_t x) { return pfx[x]; }, r.start, r.deg,
                                     (uint64_t)r.w_lo | ((uint64_t)r.w_hi << 32),
                                     (uint64_t)(e - r.start));
      const int32_t c1 = c0 < last ? c0 + 1 : last;
      const uint64_t p0 = pfx[c0], p1 = pfx[c1];
      const int32_t v0 = col[c0], v1 = col[c1];
      const VRec t0r = vrec[v0], t1r = vrec[v1];
      g[0] = make_uint4((uint32_t)p0, (uint32_t)(p0 >> 32), (uint32_t)p1, (uint32_t)(p1 >> 32));
      g[1] = make_uint4((uint32_t)v0, (uint32_t)t0r.start, (uint32_t)t0r.deg, (uint32_t)c0);
      g[2] = make_uint4((uint32_t)v1, (uint32_t)t1r.start, (uint32_t)t1r.deg, 0u);
      g[3] = make_uint4(t0r.w_lo, t0r.w_hi, t1r.w_lo, t1r.w_hi);
    }
    quad_exchange(g);
    const int64_t q = at - p;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (q + j < m) fat[4 * (q + j) + p] = g[j];
  }
}

// ---- device-wide exclusive scan (reduce tiles, scan tile sums, apply) ----
constexpr int kScanItems = 16;
constexpr int kScanTile = kBlock * kScanItems;

__global__ void __launch_bounds__(kBlock)
k_scan_reduce(const uint32_t* __restrict__ in, int64_t n, uint64_t* __restrict__ tile_sums) {
  __shared__ uint64_t red[kBlock / kWave + 1];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  uint64_t s = 0;
  for (int i = 0; i < kScanItems; ++i) {
    const int64_t idx = base + (int64_t)i * kBlock + threadIdx.x;
    if (idx < n) s += in[idx];
  }
  s = wave_sum(s);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t t = 0;
    for (int i = 0; i < kBlock / kWave; ++i) t += red[i];
    tile_sums[blockIdx.x] = t;
  }
}

// single block: exclusive scan of the tile sums in place; total at [ntiles].
// 256 threads of four sums each: a 1,024-thread block found no room beside
// a persistent kernel on another stream and waited for it to end.
constexpr int kScanPer = 4;
__global__ void __launch_bounds__(kBlock) k_scan_tiles(uint64_t* tile_sums, int64_t ntiles) {
  __shared__ uint64_t s[kBlock / kWave + 1];
  uint64_t carry = 0;
  for (int64_t base = 0; base < ntiles; base += kBlock * kScanPer) {
    const int64_t i0 = base + (int64_t)threadIdx.x * kScanPer;
    uint64_t x[kScanPer];
    uint64_t loc = 0;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
      x[j] = i0 + j < ntiles ? tile_sums[i0 + j] : 0ull;
      loc += x[j];
    }
    uint64_t tot;
    uint64_t run = carry + block_exclusive_sum<kBlock>(loc, s, &tot);
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
      if (i0 + j < ntiles) tile_sums[i0 + j] = run;
      run += x[j];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) tile_sums[ntiles] = carry;
}

// Each wave takes 1,024 consecutive items in four rounds of four per lane, so
// that its 16-byte loads and 32-byte stores are consecutive across lanes.
__global__ void __launch_bounds__(kBlock)
k_scan_apply(const uint32_t* __restrict__ in, int64_t n, const uint64_t* __restrict__ tile_sums,
             uint64_t* __restrict__ out) {
  __shared__ uint64_t wsum[kBlock / kWave];
  constexpr int kRounds = kScanItems / 4;
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const int64_t base =
      (int64_t)blockIdx.x * kScanTile + (int64_t)wid * (kWave * kScanItems) + 4 * lane;
  const bool wide = ((uintptr_t)in & 15) == 0;  // the caller's array may start anywhere
  uint32_t x[kRounds][4];
  uint64_t run[kRounds];  // items of the wave before this lane's four of the round
  uint64_t carry = 0;
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int64_t i = base + r * (4 * kWave);
    if (wide && i + 4 <= n) {
      const uint4 y = *reinterpret_cast<const uint4*>(in + i);
      x[r][0] = y.x;
      x[r][1] = y.y;
      x[r][2] = y.z;
      x[r][3] = y.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) x[r][j] = i + j < n ? in[i + j] : 0u;
    }
  }
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const uint64_t four = (uint64_t)x[r][0] + x[r][1] + x[r][2] + x[r][3];
    const uint64_t inc = wave_inclusive_sum(four);
    run[r] = carry + inc - four;
    carry += __shfl(inc, kWave - 1, kWave);
  }
  if (lane == 0) wsum[wid] = carry;
  __syncthreads();
  uint64_t before = tile_sums[blockIdx.x];
  for (int w = 0; w < wid; ++w) before += wsum[w];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int64_t i = base + r * (4 * kWave);
    uint64_t y[4];
    y[0] = before + run[r];
    y[1] = y[0] + x[r][0];
    y[2] = y[1] + x[r][1];
    y[3] = y[2] + x[r][2];
    if (i + 4 <= n) {
      ulonglong2* o = reinterpret_cast<ulonglong2*>(out + i);
      o[0] = make_ulonglong2(y[0], y[1]);
      o[1] = make_ulonglong2(y[2], y[3]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (i + j < n) out[i + j] = y[j];
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = tile_sums[gridDim.x];
}

// The whole scan of a few tiles by one work-group: one launch instead of
// three, of which each costs about 8 us between small kernels.  Two tiles:
// at four the tiles in turn take longer than the launches (an index of 11,282
// paths of 20 steps, four tiles a scan: the sample 183 us so, 166 in three).
constexpr int kScanSmallTiles = 2;
__global__ void __launch_bounds__(kBlock)
k_scan_small(const uint32_t* __restrict__ in, int64_t n, uint64_t* __restrict__ out) {
  __shared__ uint64_t s[kBlock / kWave + 1];
  uint64_t carry = 0;
  for (int64_t base = 0; base < n; base += kScanTile) {
    const int64_t i0 = base + (int64_t)threadIdx.x * kScanItems;
    uint32_t x[kScanItems];
    uint64_t loc = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      x[i] = i0 + i < n ? in[i0 + i] : 0u;
      loc += x[i];
    }
    uint64_t tot;
    uint64_t run = carry + block_exclusive_sum<kBlock>(loc, s, &tot);
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      if (i0 + i < n) out[i0 + i] = run;
      run += x[i];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) out[n] = carry;
}

inline unsigned grid_for(int64_t work, int per_block, unsigned cap = 1u << 30) {
  int64_t g = (work + per_block - 1) / per_block;
  if (g < 1) g = 1;
  if (g > (int64_t)cap) g = cap;
  return (unsigned)g;
}

}  // namespace

void launch_validate(const int32_t* row_ptr, const int32_t* col, int32_t n, int64_t m,
                     uint32_t* err, hipStream_t s) {
  const int64_t work = m > n ? m : n;
  k_validate<<<grid_for(work, kBlock * 8, 65536), kBlock, 0, s>>>(row_ptr, col, n, m, err);
}

void launch_check_symmetric(const int32_t* row_ptr, const int32_t* col, const uint32_t* w,
                            int32_t n, uint8_t* sorted, uint32_t* err, hipStream_t s) {
  const unsigned g = grid_for(n, kBlock / kWave, 65536);
  k_rows_sorted<<<g, kBlock, 0, s>>>(row_ptr, col, n, sorted);
  k_check_symmetric<<<g, kBlock, 0, s>>>(row_ptr, col, w, sorted, n, err);
}

int64_t edge_tiles(int64_t m) { return (m + kEdgeTile - 1) / kEdgeTile; }

void launch_rows(const int32_t* row_ptr, const uint64_t* sum, int32_t n, int start_all, VRec* vrec,
                 uint64_t* base, uint32_t* flags, int32_t* tile_row, uint64_t* max_w,
                 hipStream_t s) {
  k_rows<<<grid_for(n, kBlock), kBlock, 0, s>>>(row_ptr, sum, n, start_all, vrec, base, flags,
                                                tile_row, (unsigned long long*)max_w);
}

void launch_start_scatter(const uint32_t* flags, const uint64_t* pos, const VRec* vrec, int32_t n,
                          int32_t* vstart, int4* rec, hipStream_t s) {
  k_start_scatter<<<grid_for(n, kBlock), kBlock, 0, s>>>(flags, pos, vrec, n, vstart, rec);
}

void launch_edges32(const int32_t* row_ptr, const int32_t* tile_row, const uint64_t* sum,
                    const uint64_t* base, const int32_t* col, int32_t n, int64_t m, uint2* edge,
                    hipStream_t s) {
  if (m)
    k_edges32<<<(unsigned)edge_tiles(m), kBlock, 0, s>>>(row_ptr, tile_row, sum, base, col, n, m,
                                                         edge);
}

void launch_prefix64(const int32_t* row_ptr, const int32_t* tile_row, const uint64_t* sum,
                     const uint64_t* base, int32_t n, int64_t m, uint64_t* pfx, hipStream_t s) {
  if (m)
    k_prefix64<<<(unsigned)edge_tiles(m), kBlock, 0, s>>>(row_ptr, tile_row, sum, base, n, m, pfx);
}

void launch_guide32(const int32_t* row_ptr, const int32_t* tile_row, const VRec* vrec,
                    const uint2* edge, int32_t n, int64_t m, uint4* fat, hipStream_t s) {
  if (m)
    k_guide32<<<(unsigned)edge_tiles(m), kBlock, 0, s>>>(row_ptr, tile_row, vrec, edge, n, m, fat);
}

void launch_guide64(const int32_t* row_ptr, const int32_t* tile_row, const VRec* vrec,
                    const uint64_t* pfx, const int32_t* col, int32_t n, int64_t m, uint4* fat,
                    hipStream_t s) {
  if (m)
    k_guide64<<<(unsigned)edge_tiles(m), kBlock, 0, s>>>(row_ptr, tile_row, vrec, pfx, col, n, m,
                                                         fat);
}

size_t scan_temp_bytes(int64_t n) {
  const int64_t tiles = (n + kScanTile - 1) / kScanTile;
  return sizeof(uint64_t) * (size_t)(tiles + 2);
}

void launch_scan_u32_to_u64(const uint32_t* in, uint64_t* out, int64_t n, void* temp,
                            hipStream_t s) {
  int64_t tiles = (n + kScanTile - 1) / kScanTile;
  if (tiles <= kScanSmallTiles) {
    k_scan_small<<<1, kBlock, 0, s>>>(in, n, out);
    return;
  }
  uint64_t* ts = static_cast<uint64_t*>(temp);
  k_scan_reduce<<<(unsigned)tiles, kBlock, 0, s>>>(in, n, ts);
  k_scan_tiles<<<1, kBlock, 0, s>>>(ts, tiles);
  k_scan_apply<<<(unsigned)tiles, kBlock, 0, s>>>(in, n, ts, out);
}

}  // namespace panther
