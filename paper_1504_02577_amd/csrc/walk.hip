// GenerateRandomPath (Algorithm 3): one thread per path.
//
// Step 0 draws the start uniformly from the start set; step t >= 1 moves
// from v along the first CSR entry of v's row whose inclusive weight prefix
// exceeds u = floor(r_t * W_v / 2^64), which selects neighbour j with
// probability w_vj / W_v (Eq. 3).  A weightless row (start-all form only)
// keeps the walk in place.
//
// Rows whose weight sums fit 32 bits use a guide table: bucket
// b = floor(r_t * deg / 2^64) names the first edge e0 any draw of that bucket
// can select.  Its 64-byte record (one aligned line) holds e0 and the
// prefixes of the edges e0, e0+1, e0+2, and their targets with the targets'
// own {row start, degree, W}, so the usual step reads one line and already
// has the next vertex's record; only when the draw lies beyond e0+2 does the
// step scan packed {prefix, column} records and load the vertex record.
// The chosen edge is always the first whose prefix exceeds u, as in a
// bisection.
// Graphs with 64-bit row sums have records of the first two edges of a bucket;
// where their 64 bytes per entry do not fit in memory, each step bisects its
// row's prefixes.  Each path's T+1 vertices are written once as 16-byte stores.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace panther {

namespace {

constexpr int kBlock = 256;
constexpr int kScanMax = 8;  // forward steps before falling back to bisection
// Guide tables past this size are read with non-temporal loads: such a walk
// finds hardly a line twice (R = 6 to 12 n paths), and leaving the lines out of
// L2 took the R-MAT 24 walk (33 GB) from 14.0 to 13.4 ms and R-MAT 23 (16 GB)
// from 6.78 to 6.71; at R-MAT 22 (8 GB) and below both are alike (6.72 / 6.73),
// and tables that caches hold lose (10^5 paths: a quarter more time).
constexpr uint64_t kStreamBytes = (uint64_t)8 << 30;

template <int S>
__device__ __forceinline__ void store_row(int32_t* __restrict__ paths, uint64_t pid,
                                          const int32_t (&row)[S]) {
  int4* out = reinterpret_cast<int4*>(paths + pid * (uint64_t)S);
#pragma unroll
  for (int i = 0; i < S / 4; ++i)
    out[i] = make_int4(row[4 * i], row[4 * i + 1], row[4 * i + 2], row[4 * i + 3]);
}

template <bool NT>
__device__ __forceinline__ uint4 load_chunk(const uint4* p) {
  if constexpr (NT) {
    typedef uint32_t words __attribute__((ext_vector_type(4)));
    const words v = __builtin_nontemporal_load(reinterpret_cast<const words*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
  } else {
    return *p;
  }
}

// The 64-byte records of the four lanes of a quad: load j reads the record
// of lane j, 16 bytes per lane, so that a record is one request of 64
// consecutive bytes, and the transpose hands every lane the four chunks of
// its own.  (One lane reading its record with four 16-byte loads looks the
// line up four times, and with 2,048 lanes of a CU in flight the line could
// leave the caches in between: the walk read 97 bytes per record from HBM, and
// reads 66 now, starts included.)  What bounds it is the rate of scattered
// requests, about 45 per nanosecond (a plain read of 4 GiB in scattered 64-byte
// blocks reaches 49; a table of 128 MB, which the Infinity Cache holds, is no
// faster): R-MAT 24, 10^8 paths of 5 steps, 17.4 -> 13.4 ms; R-MAT 20, 10^7
// paths, 1.89 -> 1.20 ms.  Every lane of the quad must be active.
template <bool NT>
__device__ __forceinline__ void quad_records(const uint4* __restrict__ fat, uint32_t bucket,
                                             uint4 (&g)[4]) {
  const int p = threadIdx.x & 3;
  const uint32_t b0 = quad_move<0x00>(bucket), b1 = quad_move<0x55>(bucket),
                 b2 = quad_move<0xAA>(bucket), b3 = quad_move<0xFF>(bucket);
  g[0] = load_chunk<NT>(fat + 4 * (uint64_t)b0 + p);
  g[1] = load_chunk<NT>(fat + 4 * (uint64_t)b1 + p);
  g[2] = load_chunk<NT>(fat + 4 * (uint64_t)b2 + p);
  g[3] = load_chunk<NT>(fat + 4 * (uint64_t)b3 + p);
  quad_exchange(g);
}

// A choice between two values: between two chunks as a whole it would be one
// of addresses, and the record would be kept in LDS.
__device__ __forceinline__ uint32_t pick(bool c, uint32_t a, uint32_t b) { return c ? a : b; }

template <int S, bool NT>
__global__ void __launch_bounds__(kBlock)
k_walk32(const VRec* __restrict__ vrec, const uint2* __restrict__ edge,
         const uint4* __restrict__ fat, const int4* __restrict__ start_rec, int32_t nstart,
         int32_t T, uint64_t R, PhiloxKey key, int32_t* __restrict__ paths) {
  // threads past R walk too (their quads need every lane) and write nothing
  const uint64_t pid = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  int32_t row[S];
  const int4 s0 = start_rec[scale64(draw(key, pid, 0u), (uint64_t)nstart)];
  int32_t v = s0.x;
  row[0] = v;
  VRec cur = VRec{s0.y, s0.z, (uint32_t)s0.w, 0u};
#pragma unroll
  for (int t = 1; t < S; ++t) {
    if (t <= T) {
      const uint64_t r = draw(key, pid, (uint32_t)t);
      const uint32_t W = cur.w_lo;  // w_hi == 0 on this path
      const uint32_t u = (uint32_t)scale64(r, (uint64_t)W);
      // a weightless row (no bucket of its own) reads record 0 and stays
      uint4 g[4];
      quad_records<NT>(
          fat, W ? (uint32_t)(cur.start + (int32_t)scale64(r, (uint64_t)cur.deg)) : 0u, g);
      if (W != 0u) {
        // chunks: [pfx0 pfx1 pfx2 e0] [col st dg W] of e0, e0+1, e0+2
        if (u < g[0].z) {
          const bool c0 = u < g[0].x, c1 = u < g[0].y;
          v = (int32_t)pick(c0, g[1].x, pick(c1, g[2].x, g[3].x));
          cur = VRec{(int32_t)pick(c0, g[1].y, pick(c1, g[2].y, g[3].y)),
                     (int32_t)pick(c0, g[1].z, pick(c1, g[2].z, g[3].z)),
                     pick(c0, g[1].w, pick(c1, g[2].w, g[3].w)), 0u};
        } else {
          // rare: scan on from the fourth candidate, bisection after kScanMax
          int32_t e = (int32_t)g[0].w + 3;
          uint2 x = edge[e];
          int steps = 0;
          while (x.x <= u && steps < kScanMax) {
            ++e;
            x = edge[e];
            ++steps;
          }
          if (x.x <= u) {
            int32_t lo = e + 1, hi = cur.start + cur.deg - 1;
            while (lo < hi) {
              const int32_t mid = lo + ((hi - lo) >> 1);
              if (edge[mid].x > u)
                hi = mid;
              else
                lo = mid + 1;
            }
            x = edge[lo];
          }
          v = (int32_t)x.y;
          cur = vrec[v];
        }
      }
      row[t] = v;
    } else {
      row[t] = -1;
    }
  }
  if (pid < R) store_row<S>(paths, pid, row);
}

// The same walk with 64-bit prefixes (200,000 vertices of an R-MAT 18 with
// 32-bit weights, 10^6 paths of 20 steps: 2.28 ms by bisection, a dozen
// dependent reads a step, 0.47 with records).
template <int S>
__global__ void __launch_bounds__(kBlock)
k_walk64_guide(const VRec* __restrict__ vrec, const uint64_t* __restrict__ pfx,
               const int32_t* __restrict__ col, const uint4* __restrict__ fat,
               const int32_t* __restrict__ vstart, int32_t nstart, int32_t T, uint64_t R,
               PhiloxKey key, int32_t* __restrict__ paths) {
  // threads past R walk too (their quads need every lane) and write nothing
  const uint64_t pid = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  int32_t row[S];
  int32_t v = vstart[scale64(draw(key, pid, 0u), (uint64_t)nstart)];
  row[0] = v;
  VRec cur = vrec[v];
#pragma unroll
  for (int t = 1; t < S; ++t) {
    if (t <= T) {
      const uint64_t r = draw(key, pid, (uint32_t)t);
      const uint64_t W = (uint64_t)cur.w_lo | ((uint64_t)cur.w_hi << 32);
      const uint64_t u = scale64(r, W);
      uint4 g[4];
      quad_records<false>(
          fat, W ? (uint32_t)(cur.start + (int32_t)scale64(r, (uint64_t)cur.deg)) : 0u, g);
      if (W != 0) {
        // chunks: [pfx0 pfx1] [col st dg e0] [col st dg -] [W0 W1]
        const uint64_t p0 = (uint64_t)g[0].x | ((uint64_t)g[0].y << 32);
        const uint64_t p1 = (uint64_t)g[0].z | ((uint64_t)g[0].w << 32);
        if (u < p1) {
          const bool one = u >= p0;
          v = (int32_t)pick(one, g[2].x, g[1].x);
          cur = VRec{(int32_t)pick(one, g[2].y, g[1].y), (int32_t)pick(one, g[2].z, g[1].z),
                     pick(one, g[3].z, g[3].x), pick(one, g[3].w, g[3].y)};
        } else {
          // scan on from the third candidate, bisection after kScanMax
          int32_t e = (int32_t)g[1].w + 2;
          const int32_t last = cur.start + cur.deg - 1;
          for (int i = 0; i < kScanMax && pfx[e] <= u; ++i) ++e;
          if (pfx[e] <= u) {
            int32_t lo = e + 1, hi = last;
            while (lo < hi) {
              const int32_t mid = lo + ((hi - lo) >> 1);
              if (pfx[mid] > u)
                hi = mid;
              else
                lo = mid + 1;
            }
            e = lo;
          }
          v = col[e];
          cur = vrec[v];
        }
      }
      row[t] = v;
    } else {
      row[t] = -1;
    }
  }
  if (pid < R) store_row<S>(paths, pid, row);
}

template <int S>
__global__ void __launch_bounds__(kBlock)
k_walk64(const VRec* __restrict__ vrec, const uint64_t* __restrict__ pfx,
         const int32_t* __restrict__ col, const int32_t* __restrict__ vstart, int32_t nstart,
         int32_t T, uint64_t R, PhiloxKey key, int32_t* __restrict__ paths) {
  const uint64_t pid = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  if (pid >= R) return;
  int32_t row[S];
  int32_t v = vstart[scale64(draw(key, pid, 0u), (uint64_t)nstart)];
  row[0] = v;
#pragma unroll
  for (int t = 1; t < S; ++t) {
    if (t <= T) {
      const uint64_t r = draw(key, pid, (uint32_t)t);
      const VRec rec = vrec[v];
      const uint64_t W = (uint64_t)rec.w_lo | ((uint64_t)rec.w_hi << 32);
      if (W != 0) {
        const uint64_t u = scale64(r, W);
        int32_t lo = rec.start, hi = rec.start + rec.deg - 1;
        while (lo < hi) {
          const int32_t mid = lo + ((hi - lo) >> 1);
          if (pfx[mid] > u)
            hi = mid;
          else
            lo = mid + 1;
        }
        v = col[lo];
      }
      row[t] = v;
    } else {
      row[t] = -1;
    }
  }
  store_row<S>(paths, pid, row);
}

// Consecutive threads write consecutive entries of a work-group's `per` rows
// (10^7 rows of 24 bytes: 0.35 ms by the runtime's strided copy, 0.10 here).
__global__ void __launch_bounds__(kBlock)
k_pack_paths(const int32_t* __restrict__ paths, int stride, uint32_t w, int64_t rows, int per,
             int32_t* __restrict__ out) {
  const int64_t r0 = (int64_t)blockIdx.x * per;
  const uint32_t n = (uint32_t)(rows - r0 < per ? rows - r0 : per) * w;
  const int32_t* in = paths + r0 * stride;
  int32_t* to = out + r0 * w;
#pragma unroll 4
  for (uint32_t i = threadIdx.x; i < n; i += kBlock) {
    const uint32_t r = i / w;
    to[i] = in[r * (uint32_t)stride + (i - r * w)];
  }
}

}  // namespace

void launch_pack_paths(const int32_t* paths, int stride, int w, int64_t rows, int32_t* out,
                       hipStream_t s) {
  if (rows <= 0) return;
  // a thousand work-groups where the rows allow (16,000 rows of 21 in 16
  // work-groups of 1,024 rows took longer than the strided copy)
  const int per = (int)std::min<int64_t>(1024, std::max<int64_t>(16, rows / 1024));
  k_pack_paths<<<(unsigned)((rows + per - 1) / per), kBlock, 0, s>>>(paths, stride, (uint32_t)w,
                                                                     rows, per, out);
}

#define PANTHER_STRIDES(MACRO) \
  switch (stride) {            \
    case 4: MACRO(4); break;   \
    case 8: MACRO(8); break;   \
    case 16: MACRO(16); break; \
    case 32: MACRO(32); break; \
    default: MACRO(64); break; \
  }

void launch_walk64(int stride, const VRec* vrec, const uint64_t* pfx, const int32_t* col,
                   const uint4* fat, const int32_t* vstart, int32_t nstart, int32_t T, uint64_t R,
                   uint64_t seed, int32_t* paths, hipStream_t s) {
  const PhiloxKey key{(uint32_t)seed, (uint32_t)(seed >> 32)};
  const unsigned grid = (unsigned)((R + kBlock - 1) / kBlock);
  if (fat) {
#define PANTHER_W64(SS)                                                                         \
  k_walk64_guide<SS><<<grid, kBlock, 0, s>>>(vrec, pfx, col, fat, vstart, nstart, T, R, key, \
                                             paths)
    PANTHER_STRIDES(PANTHER_W64)
#undef PANTHER_W64
  } else {
#define PANTHER_W64(SS) \
  k_walk64<SS><<<grid, kBlock, 0, s>>>(vrec, pfx, col, vstart, nstart, T, R, key, paths)
    PANTHER_STRIDES(PANTHER_W64)
#undef PANTHER_W64
  }
}

void launch_walk32(int stride, const VRec* vrec, const uint2* edge, const uint4* fat, int64_t m,
                   const int4* start_rec, int32_t nstart, int32_t T, uint64_t R, uint64_t seed,
                   int32_t* paths, hipStream_t s) {
  const PhiloxKey key{(uint32_t)seed, (uint32_t)(seed >> 32)};
  const unsigned grid = (unsigned)((R + kBlock - 1) / kBlock);
  if ((uint64_t)m * 64 > kStreamBytes) {
#define PANTHER_W32(SS) \
  k_walk32<SS, true><<<grid, kBlock, 0, s>>>(vrec, edge, fat, start_rec, nstart, T, R, key, paths)
    PANTHER_STRIDES(PANTHER_W32)
#undef PANTHER_W32
  } else {
#define PANTHER_W32(SS) \
  k_walk32<SS, false><<<grid, kBlock, 0, s>>>(vrec, edge, fat, start_rec, nstart, T, R, key, paths)
    PANTHER_STRIDES(PANTHER_W32)
#undef PANTHER_W32
  }
}

}  // namespace panther
