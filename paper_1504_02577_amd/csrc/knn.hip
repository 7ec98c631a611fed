// Panther++ nearest neighbours in double precision (Sec. 3.3): for each
// query q, the k vertices v != q of smallest squared Euclidean distance
// between feature rows, ties by id.  The kd-tree of the paper indexes this
// same exact search; here every row is scanned (brute force).
//
// Arithmetic per pair: d2 = 0; for d in 0..D-1: delta = (double)theta_q[d]
// - (double)theta_v[d]; d2 = fma(delta, delta, d2) -- one fused multiply-add
// per coordinate in coordinate order.
//
// The cross-graph form takes the query rows from another graph's features
// and ranks every row of this one (no row is the query itself).
//
// A work-group takes 8 queries and a slice of the rows, four rows per thread
// per round.  Each query keeps a candidate buffer in LDS with a threshold (the
// kp-th best (d2, id) kept so far): candidates below it are appended, and a
// buffer with more than kp entries is bitonic-sorted by one wavefront and cut
// back to kp, which tightens the threshold.  The slices' kp best pairs are
// merged per query: the order is total, so any split gives the same k.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "kernels.h"

namespace panther {

namespace {

constexpr int kBlock = 256;
constexpr int kQT = 8;    // queries of a work-group's tile
constexpr int kRows = 4;  // database rows per thread and round
constexpr int kCols = 8;  // coordinates staged per step
static_assert(kQT * kRows <= 32, "one pending bit per (query, row)");

__device__ __forceinline__ void wave_sync_knn() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ bool pair_less(double a, int32_t va, double b, int32_t vb) {
  return a < b || (a == b && va < vb);
}

// Ascending bitonic sort of cnt (d2, id) pairs by one wavefront.
__device__ void wave_sort_pairs(double* d, int32_t* v, int cnt) {
  const int lane = threadIdx.x & (kWave - 1);
  int P = 2;
  while (P < cnt) P <<= 1;
  for (int i = cnt + lane; i < P; i += kWave) {
    d[i] = INFINITY;
    v[i] = 0x7FFFFFFF;
  }
  wave_sync_knn();
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = lane; i < (P >> 1); i += kWave) {
        const int lo = ((i & ~(stride - 1)) << 1) | (i & (stride - 1));  // stride: power of two
        const int hi = lo + stride;
        const bool asc = (lo & size) == 0;
        const double a = d[lo], b = d[hi];
        const int32_t x = v[lo], y = v[hi];
        if (pair_less(b, y, a, x) == asc) {
          d[lo] = b;
          d[hi] = a;
          v[lo] = y;
          v[hi] = x;
        }
      }
      wave_sync_knn();
    }
  }
}

// LDS of k_knn_fp64: the tile's query rows, kQT candidate buffers of `cap`
// pairs, the row stage.
constexpr int kStagePitch = kCols + 1;
__host__ __device__ constexpr size_t knn_scan_lds(int D, int cap) {
  return sizeof(double) * (size_t)kQT * D +
         (sizeof(double) + sizeof(int32_t)) * (size_t)kQT * cap +
         sizeof(float) * (size_t)kBlock * kRows * kStagePitch;
}
// Pairs a buffer holds (a power of two, for its sort): at least kp free
// places after every cut.
__host__ __device__ constexpr int knn_scan_cap(int kp) { return kp < 64 ? 128 : 2 * kp; }

// Bound: FP64 VALU, one subtraction and one fma per (query, row, coordinate),
// at 16 lanes per clock and SIMD.  A coordinate of the 8 queries is read from
// LDS by four broadcasts, each of the thread's four rows by one word (the rows
// are staged 8 coordinates at a time by coalesced loads), so that 64 FP64
// instructions follow eight LDS reads.  (Query coordinates as scalars waited
// for every load: 3.0 ms for the case below.)  The rows are split over grid.y
// so that few queries fill the chip too: 301 queries x 262,144 rows of 100
// coordinates took 43.1 ms on 19 work-groups that each scanned every row, and
// take 1.35 (the arithmetic alone 0.41).  Two waves per SIMD (28 spilled
// registers) beat one with 284 registers, 1.70 ms.
__global__ void __launch_bounds__(kBlock, 2)
k_knn_fp64(const float* __restrict__ theta, int32_t n, int32_t D, const float* __restrict__ qtheta,
           int32_t exclude_self, const int32_t* __restrict__ queries,
           const int32_t* __restrict__ rows, int64_t nq, int32_t kp, int32_t cap,
           double* __restrict__ part_d, int32_t* __restrict__ part_v, int32_t k,
           int32_t* __restrict__ out_ids, double* __restrict__ out_dist) {
  extern __shared__ __align__(16) char lds[];
  double* qv = reinterpret_cast<double*>(lds);               // [D][kQT]
  double* bd = qv + (size_t)kQT * D;                         // [kQT][cap]
  int32_t* bv = reinterpret_cast<int32_t*>(bd + kQT * cap);  // [kQT][cap]
  float* stage = reinterpret_cast<float*>(bv + kQT * cap);   // [kRows * kBlock][kStagePitch]
  __shared__ uint32_t cnt[kQT];
  __shared__ double tau_d[kQT];
  __shared__ int32_t tau_v[kQT];
  __shared__ int32_t qid[kQT];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const int64_t q0 = (int64_t)blockIdx.x * kQT;
  if (threadIdx.x < kQT) {
    const int i = threadIdx.x;
    qid[i] = (q0 + i < nq) ? queries[rows ? rows[q0 + i] : q0 + i] : -1;
    cnt[i] = 0u;
    tau_d[i] = INFINITY;
    tau_v[i] = 0x7FFFFFFF;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kQT * D; i += kBlock) {
    const int32_t q = qid[i / D];
    qv[(i % D) * kQT + i / D] = q >= 0 ? (double)qtheta[(int64_t)q * D + i % D] : 0.0;
  }
  // this slice's rounds of kRows * kBlock rows, interleaved over the slices
  constexpr int kRound = kRows * kBlock;
  const int64_t step = (int64_t)gridDim.y * kRound;
  // one step's coordinates: kCols lanes take the consecutive ones of one row
  constexpr int kStageLoads = kRound * kCols / kBlock;
  float next[kStageLoads];
  auto load_stage = [&](int64_t base, int d0) {
    const int c = d0 + (int)threadIdx.x % kCols;
#pragma unroll
    for (int i = 0; i < kStageLoads; ++i) {
      const int64_t v = base + i * (kBlock / kCols) + (int)threadIdx.x / kCols;
      next[i] = v < n && c < D ? theta[v * D + c] : 0.f;
    }
  };
  load_stage((int64_t)blockIdx.y * kRound, 0);
  for (int64_t base = (int64_t)blockIdx.y * kRound; base < n; base += step) {
    double acc[kRows][kQT];
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
      for (int q = 0; q < kQT; ++q) acc[r][q] = 0.0;
    for (int d0 = 0; d0 < D; d0 += kCols) {
      const int nc = D - d0 < kCols ? D - d0 : kCols;
#pragma unroll
      for (int i = 0; i < kStageLoads; ++i)
        stage[(i * (kBlock / kCols) + (int)threadIdx.x / kCols) * kStagePitch +
              (int)threadIdx.x % kCols] = next[i];
      // the loads of the next step (of the next round after the last one)
      // are in flight during this one's arithmetic
      if (d0 + kCols < D)
        load_stage(base, d0 + kCols);
      else
        load_stage(base + step, 0);
      __syncthreads();
#pragma unroll 2
      for (int d = 0; d < nc; ++d) {
        double x[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r)
          x[r] = (double)stage[(r * kBlock + threadIdx.x) * kStagePitch + d];
        double qd[kQT];
#pragma unroll
        for (int q = 0; q < kQT; q += 2) {
          const double2 y = *reinterpret_cast<const double2*>(qv + (d0 + d) * kQT + q);
          qd[q] = y.x;
          qd[q + 1] = y.y;
        }
#pragma unroll
        for (int q = 0; q < kQT; ++q) {
          const double qx = qd[q];
#pragma unroll
          for (int r = 0; r < kRows; ++r) {
            const double delta = qx - x[r];
            acc[r][q] = fma(delta, delta, acc[r][q]);
          }
        }
      }
      __syncthreads();
    }
    // candidates below their query's threshold; those that find no room wait
    // for the buffer's cut and are tested again
    uint32_t pend = 0u;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const int64_t v = base + r * kBlock + threadIdx.x;
#pragma unroll
      for (int q = 0; q < kQT; ++q) {
        const int32_t me = qid[q];
        if (v < n && me >= 0 && (!exclude_self || (int32_t)v != me) &&
            pair_less(acc[r][q], (int32_t)v, tau_d[q], tau_v[q]))
          pend |= 1u << (r * kQT + q);
      }
    }
    while (__syncthreads_or(pend != 0u)) {
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        const int32_t v = (int32_t)(base + r * kBlock + threadIdx.x);
#pragma unroll
        for (int q = 0; q < kQT; ++q) {
          const uint32_t bit = 1u << (r * kQT + q);
          if (!(pend & bit)) continue;
          if (!pair_less(acc[r][q], v, tau_d[q], tau_v[q])) {
            pend &= ~bit;
            continue;
          }
          const uint32_t pos = atomicAdd(&cnt[q], 1u);
          if (pos < (uint32_t)cap) {
            bd[q * cap + pos] = acc[r][q];
            bv[q * cap + pos] = v;
            pend &= ~bit;
          }
        }
      }
      __syncthreads();
      for (int q = wid; q < kQT; q += kBlock / kWave) {
        const int c = (int)cnt[q] < cap ? (int)cnt[q] : cap;
        // a cut waits until its buffer is three quarters full (the first one
        // only for kp pairs): one a round cost seven times the arithmetic
        if (c > kp && (c > cap - cap / 4 || tau_v[q] == 0x7FFFFFFF)) {
          wave_sort_pairs(bd + q * cap, bv + q * cap, c);
          if (lane == 0) {
            cnt[q] = (uint32_t)kp;
            tau_d[q] = bd[q * cap + kp - 1];
            tau_v[q] = bv[q * cap + kp - 1];
          }
        }
      }
    }
  }
  for (int q = wid; q < kQT; q += kBlock / kWave) {
    if (qid[q] < 0) continue;
    int c = (int)cnt[q];  // <= cap
    wave_sort_pairs(bd + q * cap, bv + q * cap, c);
    if (gridDim.y == 1) {  // every row seen: the answer itself
      const int64_t qi = rows ? (int64_t)rows[q0 + q] : q0 + q;
      for (int j = lane; j < k; j += kWave) {
        out_ids[qi * k + j] = j < c ? bv[q * cap + j] : -1;
        out_dist[qi * k + j] = j < c ? sqrt(bd[q * cap + j]) : INFINITY;
      }
      continue;
    }
    if (c > kp) c = kp;
    const int64_t o = ((q0 + q) * gridDim.y + blockIdx.y) * kp;
    for (int j = lane; j < kp; j += kWave) {
      part_d[o + j] = j < c ? bd[q * cap + j] : INFINITY;
      part_v[o + j] = j < c ? bv[q * cap + j] : 0x7FFFFFFF;
    }
  }
}

// One work-group per query: the k best of its slices' pairs (m of them, the
// missing ones (inf, INT32_MAX)), kMergeCap at a time beside the kp best so
// far.
constexpr int kMergeCap = 1024;
__global__ void __launch_bounds__(kBlock)
k_knn_merge(const double* __restrict__ part_d, const int32_t* __restrict__ part_v, int32_t m,
            int32_t kp, int32_t k, const int32_t* __restrict__ rows,
            int32_t* __restrict__ out_ids, double* __restrict__ out_dist) {
  __shared__ double sd[kMergeCap];
  __shared__ int32_t sv[kMergeCap];
  const int64_t q = blockIdx.x;
  const int64_t o = q * m;
  int kept = 0;
  for (int at = 0; at < m;) {
    const int take = m - at < kMergeCap - kept ? m - at : kMergeCap - kept;
    int P = 2;
    while (P < kept + take) P <<= 1;
    for (int j = kept + threadIdx.x; j < P; j += kBlock) {
      const bool ok = j < kept + take;
      sd[j] = ok ? part_d[o + at + j - kept] : INFINITY;
      sv[j] = ok ? part_v[o + at + j - kept] : 0x7FFFFFFF;
    }
    __syncthreads();
    for (int size = 2; size <= P; size <<= 1) {
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        for (int j = threadIdx.x; j < (P >> 1); j += kBlock) {
          const int lo = ((j & ~(stride - 1)) << 1) | (j & (stride - 1));  // stride: power of two
          const int hi = lo + stride;
          const bool asc = (lo & size) == 0;
          const double a = sd[lo], b = sd[hi];
          const int32_t x = sv[lo], y = sv[hi];
          if (pair_less(b, y, a, x) == asc) {
            sd[lo] = b;
            sd[hi] = a;
            sv[lo] = y;
            sv[hi] = x;
          }
        }
        __syncthreads();
      }
    }
    at += take;
    kept = kept + take < kp ? kept + take : kp;
  }
  const int64_t qi = rows ? (int64_t)rows[q] : q;
  for (int j = threadIdx.x; j < k; j += kBlock) {
    const bool ok = j < kept && sv[j] != 0x7FFFFFFF;
    out_ids[qi * k + j] = ok ? sv[j] : -1;
    out_dist[qi * k + j] = ok ? sqrt(sd[j]) : INFINITY;
  }
}

constexpr int kSelCap = 4096;

// Norm band of each listed query over a norm-ordered copy of the database
// (rows of norm^2 norm_s[0 .. rows), ascending, in units scaled by s; a
// stored row is within min(err, 2^-8 |x|) of its scaled row x = s theta_v,
// bfloat16 rounding each coordinate within 2^-8 relative).  A row whose
// exact distance to the query is at most d_k = sqrt(tau_d) has |x| within
// s d_k of s |theta_q|, so its stored norm lies in that interval widened by
// the rounding bound at its ends, and here also by 2^-15 (s|theta_q| +
// s d_k) for the FP32 rows, 2^-15 relative on the squared norms (FP32 sums)
// and 10^-9 on d_k (the FP64 distances).  Output: the band's rows [a, b).
__global__ void __launch_bounds__(kBlock)
k_knn_band(const float* __restrict__ qtheta, int32_t D, const int32_t* __restrict__ queries,
           const int32_t* __restrict__ rows, int64_t nr, const double* __restrict__ tau_d,
           const float* __restrict__ norm_s, int64_t nrows, double scale, double err,
           int64_t* __restrict__ band) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= nr) return;
  const float* tq = qtheta + (int64_t)queries[rows[i]] * D;
  double nq2 = 0.0;
  for (int d = 0; d < D; ++d) nq2 = fma((double)tq[d], (double)tq[d], nq2);
  const double rq = scale * sqrt(nq2), dk = scale * sqrt(tau_d[i]) * (1.0 + 1e-9);
  // a stored (bfloat16) row is within min(err, 2^-8 |x|) of its row x, and
  // x - min(err, 2^-8 x), x + min(err, 2^-8 x) both increase with x
  const double x0 = rq - dk > 0.0 ? rq - dk : 0.0, x1 = rq + dk;
  const double slack = (rq + dk) * 3.0517578125e-05;  // FP32 rows and norms
  const double lo = x0 - fmin(err, x0 * 0.00390625) - slack;
  const double hi = x1 + fmin(err, x1 * 0.00390625) + slack;
  const float lo2 = lo > 0.0 ? (float)(lo * lo * (1.0 - 3.0517578125e-05)) : -1.f;
  const float hi2 = (float)(hi * hi * (1.0 + 3.0517578125e-05));
  // first row with norm >= lo2, first row with norm > hi2
  int64_t a = 0, b = nrows;
  while (a < b) {
    const int64_t m = (a + b) >> 1;
    if (norm_s[m] < lo2) a = m + 1;
    else b = m;
  }
  int64_t e = a, f = nrows;
  while (e < f) {
    const int64_t m = (e + f) >> 1;
    if (norm_s[m] <= hi2) e = m + 1;
    else f = m;
  }
  band[2 * i] = a;
  band[2 * i + 1] = e;
}

// The band form of k_knn_range: work-group (i, g) compares listed query i
// with rows a_i + g*256 + t, stepping by G*256, of its band (vertex sid[p]).
__global__ void __launch_bounds__(kBlock)
k_knn_range_band(const float* __restrict__ theta, int32_t D, const float* __restrict__ qtheta,
                 int32_t exclude_self, const int32_t* __restrict__ queries,
                 const int32_t* __restrict__ rows, const double* __restrict__ tau_d,
                 const int32_t* __restrict__ tau_v, const int64_t* __restrict__ band,
                 const int32_t* __restrict__ sid, uint32_t cap, double* __restrict__ cand_d,
                 int32_t* __restrict__ cand_v, unsigned int* __restrict__ cand_n) {
  extern __shared__ __align__(16) char lds[];
  double* qv = reinterpret_cast<double*>(lds);  // [D]
  const int64_t i = blockIdx.x;
  const int32_t me = queries[rows[i]];
  for (int d = threadIdx.x; d < D; d += kBlock) qv[d] = (double)qtheta[(int64_t)me * D + d];
  __syncthreads();
  const double td = tau_d[i];
  const int32_t tv = tau_v[i];
  const int64_t b = band[2 * i + 1];
  const int64_t stride = (int64_t)gridDim.y * kBlock;
  for (int64_t p = band[2 * i] + (int64_t)blockIdx.y * kBlock + threadIdx.x; p < b; p += stride) {
    const int32_t v = sid[p];
    const float* row = theta + (int64_t)v * D;
    double acc = 0.0;
    for (int d = 0; d < D; ++d) {
      const double delta = qv[d] - (double)row[d];
      acc = fma(delta, delta, acc);
    }
    if ((!exclude_self || v != me) && (acc < td || (acc == td && v <= tv))) {
      const unsigned pos = atomicAdd(&cand_n[i], 1u);
      if (pos < cap) {
        cand_d[i * cap + pos] = acc;
        cand_v[i * cap + pos] = v;
      }
    }
  }
}

// One work-group per listed query: sort its candidates by (d2, id) and
// write the first k to output row rows[i].  A list that overflowed is left
// alone and its index is appended to ov_list.
__global__ void __launch_bounds__(kBlock)
k_knn_cand_select(const int32_t* __restrict__ rows, const double* __restrict__ cand_d,
                  const int32_t* __restrict__ cand_v, const unsigned int* __restrict__ cand_n,
                  uint32_t cap, int32_t k, int32_t* __restrict__ out_ids,
                  double* __restrict__ out_dist, int32_t* __restrict__ ov_list,
                  unsigned long long* __restrict__ ov_n) {
  __shared__ double sd[kSelCap];
  __shared__ int32_t sv[kSelCap];
  const int64_t i = blockIdx.x;
  const unsigned c = cand_n[i];
  const int64_t qi = rows[i];
  if (c > cap) {
    if (threadIdx.x == 0) ov_list[atomicAdd(ov_n, 1ull)] = (int32_t)qi;
    return;
  }
  int P = 2;
  while (P < (int)c) P <<= 1;
  for (int j = threadIdx.x; j < P; j += kBlock) {
    const bool ok = j < (int)c;
    sd[j] = ok ? cand_d[i * cap + j] : INFINITY;
    sv[j] = ok ? cand_v[i * cap + j] : 0x7FFFFFFF;
  }
  __syncthreads();
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int j = threadIdx.x; j < (P >> 1); j += kBlock) {
        const int lo = ((j & ~(stride - 1)) << 1) | (j & (stride - 1));  // stride: power of two
        const int hi = lo + stride;
        const bool asc = (lo & size) == 0;
        const double a = sd[lo], b = sd[hi];
        const int32_t x = sv[lo], y = sv[hi];
        if (pair_less(b, y, a, x) == asc) {
          sd[lo] = b;
          sd[hi] = a;
          sv[lo] = y;
          sv[hi] = x;
        }
      }
      __syncthreads();
    }
  }
  for (int j = threadIdx.x; j < k; j += kBlock) {
    const bool ok = j < (int)c;
    out_ids[qi * k + j] = ok ? sv[j] : -1;
    out_dist[qi * k + j] = ok ? sqrt(sd[j]) : INFINITY;
  }
}

}  // namespace

size_t knn_range_bytes(int64_t nr) {
  return (sizeof(double) + sizeof(int32_t)) * (size_t)nr * kSelCap + sizeof(unsigned) * nr +
         sizeof(int32_t) * nr + 2 * sizeof(int64_t) * nr + 256;
}

// Exact recompute of listed queries from a known bound: rows[i] (i < nr)
// names the output row of query queries[rows[i]], and (tau_d[i], tau_v[i])
// is an exact (d2, id) pair that at least k rows reach.  work: device
// memory of knn_range_bytes(nr) bytes; nb: the norm-ordered copy whose
// band of each query is scanned.  A list keeps up to min(cap, 4096)
// candidates; lists that outgrow it are recomputed by the full brute force
// (one host synchronisation).
int launch_knn_recompute(const float* theta, int32_t n, int32_t D, const float* qtheta,
                         bool exclude_self, const int32_t* queries, const int32_t* rows,
                         int64_t nr, const double* tau_d, const int32_t* tau_v, int32_t k,
                         int num_cus, void* work, unsigned long long* ov_n_dev,
                         int32_t* out_ids, double* out_dist, hipStream_t s, uint32_t cap,
                         const KnnBand* nb) {
  cap = std::min<uint32_t>(cap, kSelCap);
  if (nr <= 0) return 0;
  if (!nb) return (int)hipErrorInvalidValue;
  char* w = static_cast<char*>(work);
  double* cand_d = reinterpret_cast<double*>(w);
  int32_t* cand_v = reinterpret_cast<int32_t*>(cand_d + (size_t)nr * kSelCap);
  int64_t* band = reinterpret_cast<int64_t*>(cand_v + (size_t)nr * kSelCap);  // 8-aligned
  unsigned* cand_n = reinterpret_cast<unsigned*>(band + 2 * nr);
  int32_t* ov_list = reinterpret_cast<int32_t*>(cand_n + nr);
  hipError_t e = hipMemsetAsync(cand_n, 0, sizeof(unsigned) * nr, s);
  if (e != hipSuccess) return (int)e;
  e = hipMemsetAsync(ov_n_dev, 0, sizeof(unsigned long long), s);
  if (e != hipSuccess) return (int)e;
  {
    // rows in the norm order of a sorted copy, each query within its band
    k_knn_band<<<(unsigned)((nr + kBlock - 1) / kBlock), kBlock, 0, s>>>(
        qtheta, D, queries, rows, nr, tau_d, nb->norm_s, nb->rows, nb->scale, nb->err, band);
    e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    // at least 64 work-groups per query (up to 256 for a few queries):
    // bands differ by orders of magnitude (a hub's spans most rows), and
    // the work-groups of a narrow band find nothing to do and end at once
    const int64_t gy = std::max<int64_t>(
        64, std::min<int64_t>(256, (4 * (int64_t)num_cus + nr - 1) / nr));
    const size_t lds = sizeof(double) * D;
    k_knn_range_band<<<dim3((unsigned)nr, (unsigned)gy), kBlock, lds, s>>>(
        theta, D, qtheta, exclude_self ? 1 : 0, queries, rows, tau_d, tau_v, band, nb->sid, cap,
        cand_d, cand_v, cand_n);
    e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
  }
  k_knn_cand_select<<<(unsigned)nr, kBlock, 0, s>>>(rows, cand_d, cand_v, cand_n, cap, k,
                                                   out_ids, out_dist, ov_list, ov_n_dev);
  e = hipGetLastError();
  if (e != hipSuccess) return (int)e;
  unsigned long long ov = 0;
  e = hipMemcpyAsync(&ov, ov_n_dev, sizeof ov, hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return (int)e;
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return (int)e;
  if (ov == 0) return 0;
  // the candidate lists are done with: their place (48 KiB per listed query,
  // more than one slice needs) is the scan's
  return launch_knn_fp64(theta, n, D, qtheta, exclude_self, queries, ov_list, (int64_t)ov, k,
                         num_cus, work, (sizeof(double) + sizeof(int32_t)) * (size_t)nr * kSelCap,
                         out_ids, out_dist, s);
}

namespace {
// Workspace of the FP64 form: per query S slices of kp pairs (one slice
// writes the results itself).
size_t fp64_bytes(int64_t nq, int64_t S, int kp) {
  return S > 1 ? (sizeof(double) + sizeof(int32_t)) * (size_t)nq * S * kp : 0;
}
int pow2_at_least(int k) {
  int kp = 1;
  while (kp < k) kp <<= 1;
  return kp;
}
// Slices of the rows: as many as give the two work-groups that a CU holds
// (about 60 KB of LDS each) without starting a third, where the queries' tiles
// alone are fewer; each with at least four rounds of rows, and at most 4,096
// pairs per query to merge.
int64_t fp64_slices(int64_t nq, int32_t n, int kp, int num_cus) {
  const int64_t tiles = (nq + kQT - 1) / kQT;
  int64_t S = 2 * (int64_t)num_cus / tiles;
  S = std::min<int64_t>(S, (n + 4 * kRows * kBlock - 1) / (4 * kRows * kBlock));
  S = std::min<int64_t>(S, 4096 / kp);
  return std::max<int64_t>(S, 1);
}
}  // namespace

size_t knn_fp64_bytes(int64_t nq, int32_t n, int32_t k, int num_cus) {
  if (nq <= 0) return 0;
  const int kp = pow2_at_least(k);
  return fp64_bytes(nq, fp64_slices(nq, n, kp, num_cus), kp);
}

// qtheta: the queries' feature rows (theta itself for one graph, the other
// graph's for the cross-graph form, which excludes no row).  rows (may be
// null): the call answers queries[rows[i]] into output row rows[i] for
// i < nq, instead of queries[i] into row i.  work: knn_fp64_bytes(nq, ...)
// bytes (up to 12 MiB), or less, or none: then in fewer slices.
int launch_knn_fp64(const float* theta, int32_t n, int32_t D, const float* qtheta,
                    bool exclude_self, const int32_t* queries, const int32_t* rows, int64_t nq,
                    int32_t k, int num_cus, void* work, size_t work_bytes, int32_t* out_ids,
                    double* out_dist, hipStream_t s) {
  const int kp = pow2_at_least(k);
  const int cap = knn_scan_cap(kp);
  const size_t lds = knn_scan_lds(D, cap);
  hipError_t e = hipFuncSetAttribute((const void*)k_knn_fp64,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return (int)e;
  if (nq <= 0) return 0;
  int64_t S = fp64_slices(nq, n, kp, num_cus);
  while (S > 1 && fp64_bytes(nq, S, kp) > work_bytes) --S;
  double* part_d = static_cast<double*>(work);
  int32_t* part_v = S > 1 ? reinterpret_cast<int32_t*>(part_d + nq * S * kp) : nullptr;
  k_knn_fp64<<<dim3((unsigned)((nq + kQT - 1) / kQT), (unsigned)S), kBlock, lds, s>>>(
      theta, n, D, qtheta, exclude_self ? 1 : 0, queries, rows, nq, kp, cap, part_d, part_v, k,
      out_ids, out_dist);
  if (S > 1)
    k_knn_merge<<<(unsigned)nq, kBlock, 0, s>>>(part_d, part_v, (int32_t)(S * kp), kp, k, rows,
                                                out_ids, out_dist);
  return (int)hipGetLastError();
}

}  // namespace panther
