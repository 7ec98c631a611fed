// C ABI and host runtime of the Panther library: context, device memory,
// argument validation, and the sequencing of the kernels of each call.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/panther.h"
#include "common.h"
#include "kernels.h"
#include "runtime.h"

using namespace panther;

// ---------------------------------------------------------------------------
// errors and allocation
// ---------------------------------------------------------------------------
int ctx_fail(panther_ctx* c, int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (c) {
    std::lock_guard<std::mutex> g(c->err_mu);
    c->err = buf;
  }
  return code;
}

int ctx_hip(panther_ctx* c, hipError_t e, const char* what) {
  if (e == hipSuccess) return PANTHER_OK;
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    return ctx_fail(c, PANTHER_ENOMEM, "%s: out of device memory", what);
  }
  return ctx_fail(c, PANTHER_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

// Frees memory the context holds but can do without, for an allocation that
// failed: first what only a repeat of an earlier call would use again, then
// the guide records of a graph with 64-bit row sums, which is walked by
// bisection from then on.  False once nothing is left to free.
static bool give_back(panther_ctx* c) {
  std::lock_guard<std::mutex> g(c->spare_mu);
  bool any = false;
  auto drop = [&](DevBuf& b) {
    if (!b.p) return;
    ctx_release(b);  // (hipFree waits for the kernels that use it)
    any = true;
  };
  drop(c->lane0.b_seen);  // an earlier call's: query_lengths drops its own before it asks for more
  if (!c->has_graph) return any;
  for (DevBuf* b : {&c->g_flags, &c->g_spos, &c->g_base, &c->g_tiles, &c->g_scan}) drop(*b);
  if (!any && c->pfx64 && c->d_fat) {
    c->d_fat = nullptr;
    drop(c->g_fat);
  }
  return any;
}

int ctx_alloc(panther_ctx* c, void** p, size_t bytes, const char* what) {
  *p = nullptr;
  bool inject = false;
  {
    std::lock_guard<std::mutex> g(c->alloc_mu);
    if (c->fail_alloc_after == 0)
      inject = true;
    else if (c->fail_alloc_after > 0)
      --c->fail_alloc_after;
  }
  if (inject) {
    if (!what) return PANTHER_ENOMEM;
    return ctx_fail(c, PANTHER_ENOMEM, "%s: allocation failure injected", what);
  }
  if (bytes == 0) bytes = 16;
  auto device_alloc = [&] {
    const bool room = !c->mem_reserve || device_room(c) >= bytes;
    return room ? hipMalloc(p, bytes) : hipErrorOutOfMemory;
  };
  hipError_t e = device_alloc();
  while (e != hipSuccess && give_back(c)) {
    (void)hipGetLastError();
    e = device_alloc();
  }
  if (e != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    if (!what) return PANTHER_ENOMEM;
    return ctx_fail(c, PANTHER_ENOMEM, "%s: cannot allocate %zu bytes", what, bytes);
  }
  return PANTHER_OK;
}

size_t device_room(panther_ctx* c) {
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  const size_t keep = (size_t)c->mem_reserve;
  return free_b > keep ? free_b - keep : 0;
}

void ctx_free(void* p) {
  if (p) (void)hipFree(p);
}

int ctx_ensure(panther_ctx* c, DevBuf& b, size_t bytes, const char* what) {
  if (bytes <= b.cap && b.p) return PANTHER_OK;
  ctx_free(b.p);
  b.p = nullptr;
  b.cap = 0;
  void* p;
  const int st = ctx_alloc(c, &p, bytes, what);
  if (st) return st;
  b.p = p;
  b.cap = bytes;
  return PANTHER_OK;
}

void ctx_release(DevBuf& b) {
  ctx_free(b.p);
  b.p = nullptr;
  b.cap = 0;
}

int pinned_ensure(panther_ctx* c, PinnedBuf& b, size_t bytes, const char* what) {
  if (bytes <= b.cap && b.p) return PANTHER_OK;
  pinned_release(b);
  void* p = nullptr;
  if (hipHostMalloc(&p, bytes < 4096 ? 4096 : bytes, hipHostMallocDefault) != hipSuccess || !p)
    return ctx_fail(c, PANTHER_ENOMEM, "out of pinned host memory (%s)", what);
  b.p = p;
  b.cap = bytes < 4096 ? 4096 : bytes;
  return PANTHER_OK;
}

void pinned_release(PinnedBuf& b) {
  if (b.p) (void)hipHostFree(b.p);
  b.p = nullptr;
  b.cap = 0;
}


static void free_features(panther_ctx* c) {
  ctx_free(c->d_theta);
  c->d_theta = nullptr;
  c->theta_D = 0;
  free_pp_state(c);
}

// Drops the paths, index and everything derived from them.  The storage of
// the paths and index is kept for the next sample_paths call unless
// `release` is set (a new graph, or destroy).
static void free_paths(panther_ctx* c, bool release) {
  free_features(c);
  forget_batch_graph(&c->lane0);
  c->d_paths = nullptr;
  c->d_inv_ptr = nullptr;
  c->d_inv_pid = nullptr;
  c->has_paths = false;
  c->nnz = 0;
  if (release) {
    free_lane(&c->lane0);
    for (DevBuf* b : {&c->b_paths, &c->b_inv_pid, &c->b_inv_ptr, &c->b_keys0, &c->b_keys1,
                      &c->b_vtmp, &c->b_hist, &c->b_offs, &c->b_stemp, &c->b_nnz, &c->b_allv, &c->b_queries,
                      &c->b_outs})
      ctx_release(*b);
    ctx_free(c->d_cnt);
    ctx_free(c->d_touched);
    ctx_free(c->d_ctl);
    c->d_cnt = nullptr;
    c->d_touched = nullptr;
    c->d_ctl = nullptr;
  }
}

// Storage of the graph and of its preparation, kept for the next load_graph
// (an R-MAT 22 load allocates 10 GB, which took up to 0.3 s of it).
static DevBuf panther_ctx::*const kGraphBuffers[] = {
    &panther_ctx::g_col,  &panther_ctx::g_vrec, &panther_ctx::g_pfx,  &panther_ctx::g_vstart,
    &panther_ctx::g_edge, &panther_ctx::g_fat,  &panther_ctx::g_srec, &panther_ctx::g_flags,
    &panther_ctx::g_spos, &panther_ctx::g_base, &panther_ctx::g_tiles, &panther_ctx::g_scan,
    &panther_ctx::g_ctl};

// Drops the graph and everything sampled from it; `release` gives the
// graph's storage back too.
static void free_graph(panther_ctx* c, bool release) {
  free_paths(c, true);
  c->d_edge = nullptr;
  c->d_fat = nullptr;
  c->d_start_rec = nullptr;
  c->d_col = nullptr;
  c->d_vrec = nullptr;
  c->d_pfx = nullptr;
  c->d_vstart = nullptr;
  c->has_graph = false;
  if (release)
    for (DevBuf panther_ctx::*b : kGraphBuffers) ctx_release(c->*b);
}

// A graph buffer of at least `bytes`: the kept one unless it is too small, or
// more than 64 MiB and a sixteenth too large (graphs of about one size share
// their storage; else what a graph holds, and whether there is room for
// optional records, is not to depend on the graphs before it).
template <typename T>
static int graph_alloc(panther_ctx* c, DevBuf& b, size_t bytes, const char* what, T** out) {
  if (b.cap > bytes + std::max(bytes / 16, (size_t)64 << 20)) ctx_release(b);
  const int st = ctx_ensure(c, b, std::max<size_t>(bytes, 16), what);
  *out = st ? nullptr : static_cast<T*>(b.p);
  return st;
}

// RAII holder for temporaries of a call
struct Temp {
  std::vector<void*> ptrs;
  ~Temp() {
    for (void* p : ptrs) ctx_free(p);
  }
  void* add(void* p) {
    ptrs.push_back(p);
    return p;
  }
};

void stage_begin(panther_ctx* c, int stage, hipStream_t s) {
  if (!c->timing) return;
  if (!c->ev[0]) {
    for (int i = 0; i < 10; ++i) (void)hipEventCreate(&c->ev[i]);
  }
  (void)hipEventRecord(c->ev[2 * stage], s);
}

void stage_end(panther_ctx* c, int stage, hipStream_t s) {
  if (!c->timing) return;
  (void)hipEventRecord(c->ev[2 * stage + 1], s);
  c->ev_used[stage] = true;
}

extern "C" int panther_stage_times(panther_ctx* c, double* out_ms) {
  if (!c || !out_ms) return PANTHER_EINVAL;
  if (!c->timing) return ctx_fail(c, PANTHER_ESTATE, "timing option is off");
  for (int i = 0; i < 5; ++i) {
    out_ms[i] = -1.0;
    if (!c->ev_used[i]) continue;
    float ms = 0.f;
    if (hipEventSynchronize(c->ev[2 * i + 1]) != hipSuccess ||
        hipEventElapsedTime(&ms, c->ev[2 * i], c->ev[2 * i + 1]) != hipSuccess) {
      (void)hipGetLastError();
      continue;
    }
    out_ms[i] = ms;
  }
  return PANTHER_OK;
}

int order_begin(panther_ctx* c, hipStream_t s) {
  if (!c->order_ev) {
    HIPTRY(hipEventCreateWithFlags(&c->order_ev, hipEventDisableTiming), "order event");
  }
  if (c->order_pending) HIPTRY(hipStreamWaitEvent(s, c->order_ev, 0), "order wait");
  return PANTHER_OK;
}

int order_end(panther_ctx* c, hipStream_t s) {
  HIPTRY(hipEventRecord(c->order_ev, s), "order record");
  c->order_pending = true;
  return PANTHER_OK;
}

static hipStream_t pick_stream(panther_ctx* c, void* s) {
  return s ? static_cast<hipStream_t>(s) : c->stream;
}

// ---------------------------------------------------------------------------
// create / destroy / errors / options
// ---------------------------------------------------------------------------
extern "C" int panther_create(int device_ordinal, panther_ctx** out) {
  if (!out) return PANTHER_EINVAL;
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device_ordinal < 0 || device_ordinal >= ndev) {
    (void)hipGetLastError();
    return PANTHER_EINVAL;
  }
  if (hipSetDevice(device_ordinal) != hipSuccess) return PANTHER_EDEVICE;
  panther_ctx* c = new panther_ctx();
  c->device = device_ordinal;
  if (hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking) != hipSuccess) {
    delete c;
    return PANTHER_EDEVICE;
  }
  // the cross-stream ordering event exists from the start, so that no query
  // call (the allocation-free one included) creates driver objects
  if (hipEventCreateWithFlags(&c->order_ev, hipEventDisableTiming) != hipSuccess) {
    (void)hipStreamDestroy(c->stream);
    delete c;
    return PANTHER_EDEVICE;
  }
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device_ordinal) == hipSuccess) {
    c->num_cus = prop.multiProcessorCount;
    c->lds_per_block = (int)prop.sharedMemPerBlock;
  }
  *out = c;
  return PANTHER_OK;
}

extern "C" void panther_destroy(panther_ctx* c) {
  if (!c) return;
  (void)hipSetDevice(c->device);
  (void)hipStreamSynchronize(c->stream);
  free_graph(c, true);
  for (int i = 0; i < 10; ++i)
    if (c->ev[i]) (void)hipEventDestroy(c->ev[i]);
  if (c->order_ev) (void)hipEventDestroy(c->order_ev);
  (void)hipStreamDestroy(c->stream);
  delete c;
}

extern "C" const char* panther_last_error(const panther_ctx* c) {
  return c ? c->err.c_str() : "null context";
}

extern "C" int panther_set_option(panther_ctx* c, const char* key, int64_t value) {
  if (!c || !key) return PANTHER_EINVAL;
  std::string k(key);
  if (k == "topk.form") {
    if (value != PANTHER_FORM_PLAIN && value != PANTHER_FORM_BATCHED)
      return ctx_fail(c, PANTHER_EINVAL, "topk.form must be 0 (plain) or 1 (batched)");
    c->topk_form = (int)value;
  } else if (k == "pp.form") {
    if (value != PANTHER_PP_FP64 && value != PANTHER_PP_BF16)
      return ctx_fail(c, PANTHER_EINVAL, "pp.form must be 0 (fp64) or 1 (bf16)");
    c->pp_form = (int)value;
  } else if (k == "pp.pool") {
    if (value < 32 || value > 1024)
      return ctx_fail(c, PANTHER_EINVAL, "pp.pool must lie in [32, 1024]");
    c->pp_pool = (int)value;
  } else if (k == "pp.qw") {
    if (value != 0 && value != 16 && value != 32 && value != 64)
      return ctx_fail(c, PANTHER_EINVAL, "pp.qw must be 0 (tuned), 16, 32 or 64");
    c->pp_qw = (int)value;
  } else if (k == "autotune") {
    if (value != 0 && value != 1) return ctx_fail(c, PANTHER_EINVAL, "autotune must be 0 or 1");
    c->autotune = (int)value;
  } else if (k == "timing") {
    if (value != 0 && value != 1) return ctx_fail(c, PANTHER_EINVAL, "timing must be 0 or 1");
    c->timing = (int)value;
    for (int i = 0; i < 5; ++i) c->ev_used[i] = false;
  } else if (k == "test.pp_recompute_all") {
    if (value < 0 || value > 2)
      return ctx_fail(c, PANTHER_EINVAL, "test.pp_recompute_all must be 0, 1 or 2");
    c->pp_recompute_all = (int)value;
  } else if (k == "test.fail_alloc_after") {
    c->fail_alloc_after = value < 0 ? -1 : value;
  } else if (k == "test.mem_reserve") {
    if (value < 0) return ctx_fail(c, PANTHER_EINVAL, "test.mem_reserve must be >= 0");
    c->mem_reserve = value;
  } else if (k == "batch.tier_a" || k == "batch.tier_b" || k == "batch.block" ||
             k == "batch.wgs_per_cu" || k == "batch.hub_bits" || k == "batch.tier_b_div" ||
             k == "batch.bucket_bias" || k == "test.hub_budget") {
    return set_batch_option(c, k, value);
  } else {
    return ctx_fail(c, PANTHER_EINVAL, "unknown option '%s'", key);
  }
  return PANTHER_OK;
}

extern "C" int64_t panther_sample_size(double eps, double cc, double delta, int32_t T) {
  if (!(eps > 0.0 && eps < 1.0) || !(delta > 0.0 && delta < 1.0) || !(cc > 0.0) || T < 2)
    return PANTHER_EINVAL;
  const double pairs = 0.5 * (double)T * (double)(T - 1);
  const double r = cc / (eps * eps) * (std::log2(pairs) + 1.0 + std::log(1.0 / delta));
  return (int64_t)std::ceil(r);
}

extern "C" int panther_synchronize(panther_ctx* c) {
  if (!c) return PANTHER_EINVAL;
  return ctx_hip(c, hipStreamSynchronize(c->stream), "synchronize");
}

// ---------------------------------------------------------------------------
// load_graph (a1): validate, W_v, start set, per-row prefixes
// ---------------------------------------------------------------------------
// records: with guide records where they fit.  Without, a graph with 64-bit
// row sums takes no more than its bisection form needs, and one with narrow
// sums, which is walked by records only, ends with ENOMEM.
static int load_graph(panther_ctx* c, int32_t n, int64_t m, const int32_t* row_ptr,
                      const int32_t* col, const uint32_t* w, int mem, uint32_t flags,
                      bool records) {
  if (hipSetDevice(c->device) != hipSuccess) return ctx_fail(c, PANTHER_EDEVICE, "hipSetDevice");
  if (n < 1) return ctx_fail(c, PANTHER_EINVAL, "n must be >= 1");
  if (m < 0 || m >= (int64_t(1) << 31))
    return ctx_fail(c, PANTHER_EINVAL, "m must lie in [0, 2^31)");
  if (!row_ptr || (m > 0 && (!col || !w)))
    return ctx_fail(c, PANTHER_EINVAL, "null CSR pointer");
  if (mem != PANTHER_MEM_HOST && mem != PANTHER_MEM_DEVICE)
    return ctx_fail(c, PANTHER_EINVAL, "mem must be PANTHER_MEM_HOST or PANTHER_MEM_DEVICE");
  if (flags & ~(PANTHER_START_ALL_VERTICES | PANTHER_CHECK_SYMMETRIC))
    return ctx_fail(c, PANTHER_EINVAL, "unknown flags");
  hipStream_t s = c->stream;
  int32_t ends[2];
  if (mem == PANTHER_MEM_HOST) {
    ends[0] = row_ptr[0];
    ends[1] = row_ptr[n];
  } else {
    HIPTRY(hipMemcpyAsync(&ends[0], row_ptr, 4, hipMemcpyDeviceToHost, s), "load_graph");
    HIPTRY(hipMemcpyAsync(&ends[1], row_ptr + n, 4, hipMemcpyDeviceToHost, s), "load_graph");
    HIPTRY(hipStreamSynchronize(s), "load_graph");
  }
  if (ends[0] != 0 || (int64_t)ends[1] != m)
    return ctx_fail(c, PANTHER_EINVAL, "row_ptr must start at 0 and end at m");

  free_graph(c, false);
  Temp tmp;
  const int32_t* d_rp = row_ptr;
  const uint32_t* d_w = w;
  void* p;
  TRY(graph_alloc(c, c->g_col, sizeof(int32_t) * (size_t)m, "graph columns", &c->d_col));
  int32_t* d_col = c->d_col;
  if (mem == PANTHER_MEM_HOST) {
    TRY(ctx_alloc(c, &p, sizeof(int32_t) * (size_t)(n + 1), "row_ptr staging"));
    tmp.add(p);
    HIPTRY(hipMemcpyAsync(p, row_ptr, sizeof(int32_t) * (size_t)(n + 1), hipMemcpyHostToDevice, s),
           "row_ptr upload");
    d_rp = static_cast<const int32_t*>(p);
    TRY(ctx_alloc(c, &p, sizeof(uint32_t) * (size_t)m, "weight staging"));
    tmp.add(p);
    if (m)
      HIPTRY(hipMemcpyAsync(p, w, sizeof(uint32_t) * (size_t)m, hipMemcpyHostToDevice, s),
             "weight upload");
    d_w = static_cast<const uint32_t*>(p);
    if (m)
      HIPTRY(hipMemcpyAsync(d_col, col, sizeof(int32_t) * (size_t)m, hipMemcpyHostToDevice, s),
             "column upload");
  } else if (m) {
    HIPTRY(hipMemcpyAsync(d_col, col, sizeof(int32_t) * (size_t)m, hipMemcpyDeviceToDevice, s),
           "column copy");
  }
  // small control block: [0] error bits, [2..3] max W (u64)
  uint32_t* ctl;
  TRY(graph_alloc(c, c->g_ctl, 64, "control", &ctl));
  HIPTRY(hipMemsetAsync(ctl, 0, 64, s), "control clear");
  launch_validate(d_rp, d_col, n, m, ctl, s);
  HIPTRY(hipGetLastError(), "validate");
  uint32_t hctl[4];
  HIPTRY(hipMemcpyAsync(hctl, ctl, 16, hipMemcpyDeviceToHost, s), "validate");
  HIPTRY(hipStreamSynchronize(s), "validate");
  if (hctl[0] & 1u) {
    free_graph(c, false);
    return ctx_fail(c, PANTHER_EINVAL, "row_ptr decreases");
  }
  if (hctl[0] & 2u) {
    free_graph(c, false);
    return ctx_fail(c, PANTHER_EINVAL, "column id out of range");
  }
  if (flags & PANTHER_CHECK_SYMMETRIC) {
    TRY(ctx_alloc(c, &p, (size_t)n, "row order flags"));
    tmp.add(p);
    launch_check_symmetric(d_rp, d_col, d_w, n, static_cast<uint8_t*>(p), ctl, s);
    HIPTRY(hipGetLastError(), "symmetry check");
    HIPTRY(hipMemcpyAsync(hctl, ctl, 16, hipMemcpyDeviceToHost, s), "symmetry check");
    HIPTRY(hipStreamSynchronize(s), "symmetry check");
    if (hctl[0] & 4u) {
      free_graph(c, false);
      return ctx_fail(c, PANTHER_EINVAL,
                      "CSR is not symmetric: an entry v->u of weight w lacks a matching u->v "
                      "of weight w");
    }
  }
  TRY(graph_alloc(c, c->g_vrec, sizeof(VRec) * (size_t)n, "vertex records", &c->d_vrec));
  // The scan of the weights goes where the guide records will be (written
  // last), or, when those do not fit, where the 64-bit prefixes of a graph
  // with wide row sums will be (shifted by one entry, in place).
  // (At least one record: the walk reads record 0 at weightless vertices.)
  uint64_t* sum = nullptr;
  const size_t fat_bytes = 4 * sizeof(uint4) * (size_t)std::max<int64_t>(m, 1);
  if (records && graph_alloc(c, c->g_fat, fat_bytes, "guide records", &c->d_fat) == PANTHER_OK) {
    sum = reinterpret_cast<uint64_t*>(c->d_fat);
  } else {
    TRY(graph_alloc(c, c->g_pfx, sizeof(uint64_t) * (size_t)(m + 1), "weight prefixes", &sum));
    c->d_pfx = sum;
  }
  const int start_all = (flags & PANTHER_START_ALL_VERTICES) ? 1 : 0;
  uint32_t* sflags;
  uint64_t *spos, *base;
  int32_t* tile_row;
  char* stemp;
  TRY(graph_alloc(c, c->g_flags, sizeof(uint32_t) * (size_t)n, "start flags", &sflags));
  TRY(graph_alloc(c, c->g_spos, sizeof(uint64_t) * (size_t)(n + 1), "start positions", &spos));
  TRY(graph_alloc(c, c->g_base, sizeof(uint64_t) * (size_t)n, "row offsets", &base));
  TRY(graph_alloc(c, c->g_tiles, sizeof(int32_t) * (size_t)(edge_tiles(m) + 1), "tile rows",
                  &tile_row));
  TRY(graph_alloc(c, c->g_scan, scan_temp_bytes(std::max<int64_t>(n, m)), "scan temp", &stemp));
  launch_scan_u32_to_u64(d_w, sum, m, stemp, s);
  launch_rows(d_rp, sum, n, start_all, c->d_vrec, base, sflags, tile_row,
              reinterpret_cast<uint64_t*>(ctl + 2), s);
  launch_scan_u32_to_u64(sflags, spos, n, stemp, s);
  HIPTRY(hipGetLastError(), "row sums");
  uint64_t nstart = 0;
  HIPTRY(hipMemcpyAsync(hctl, ctl, 16, hipMemcpyDeviceToHost, s), "row sums");
  HIPTRY(hipMemcpyAsync(&nstart, spos + n, 8, hipMemcpyDeviceToHost, s), "start set");
  HIPTRY(hipStreamSynchronize(s), "row sums");
  const uint64_t max_w = (uint64_t)hctl[2] | ((uint64_t)hctl[3] << 32);
  if (max_w >= (uint64_t(1) << 63)) {
    free_graph(c, false);
    return ctx_fail(c, PANTHER_EINVAL, "row weight sum exceeds 2^63");
  }
  if (nstart == 0) {
    free_graph(c, false);
    return ctx_fail(c, PANTHER_EINVAL, "no vertex has an edge of positive weight");
  }
  c->pfx64 = max_w >= (uint64_t(1) << 32);
  if (!c->pfx64 && !c->d_fat)
    return ctx_fail(c, PANTHER_ENOMEM, "guide records: cannot allocate %zu bytes", fat_bytes);
  TRY(graph_alloc(c, c->g_vstart, sizeof(int32_t) * (size_t)nstart, "start set", &c->d_vstart));
  if (!c->pfx64)
    TRY(graph_alloc(c, c->g_srec, sizeof(int4) * (size_t)nstart, "start records",
                    &c->d_start_rec));
  launch_start_scatter(sflags, spos, c->d_vrec, n, c->d_vstart, c->d_start_rec, s);
  if (c->pfx64) {
    ctx_release(c->g_edge);  // storage of a graph with narrow row sums
    ctx_release(c->g_srec);
    if (!c->d_pfx)
      TRY(graph_alloc(c, c->g_pfx, sizeof(uint64_t) * (size_t)(m + 1), "weight prefixes",
                      &c->d_pfx));
    launch_prefix64(d_rp, tile_row, sum, base, n, m, c->d_pfx + 1, s);
    // guide records only where they leave at least as much memory free as
    // they take: such a graph has to load, and leave room for its paths, in
    // as little memory as the bisection form needs
    if (c->d_fat && device_room(c) < fat_bytes) {
      HIPTRY(hipStreamSynchronize(s), "prefix");
      ctx_release(c->g_fat);
      c->d_fat = nullptr;
    }
    if (c->d_fat) launch_guide64(d_rp, tile_row, c->d_vrec, c->d_pfx + 1, d_col, n, m, c->d_fat, s);
  } else {
    ctx_release(c->g_pfx);
    TRY(graph_alloc(c, c->g_edge, sizeof(uint2) * (size_t)m, "packed edges", &c->d_edge));
    launch_edges32(d_rp, tile_row, sum, base, d_col, n, m, c->d_edge, s);
    launch_guide32(d_rp, tile_row, c->d_vrec, c->d_edge, n, m, c->d_fat, s);
  }
  HIPTRY(hipGetLastError(), "prefix");
  HIPTRY(hipStreamSynchronize(s), "load_graph");
  c->n = n;
  c->m = m;
  c->nstart = (int32_t)nstart;
  c->max_w = max_w;
  c->has_graph = true;
  return PANTHER_OK;
}

extern "C" int panther_load_graph(panther_ctx* c, int32_t n, int64_t m, const int32_t* row_ptr,
                                  const int32_t* col, const uint32_t* w, int mem,
                                  uint32_t flags) {
  if (!c) return PANTHER_EINVAL;
  c->err.clear();
  bool kept = false;
  for (DevBuf panther_ctx::*b : kGraphBuffers) kept = kept || (c->*b).p;
  int st = load_graph(c, n, m, row_ptr, col, w, mem, flags, true);
  // short of memory: once more without the previous graph's storage, which
  // may hold what is missing, then without the optional records
  for (const bool records : {true, false}) {
    if (st != PANTHER_ENOMEM) break;
    if (records && !kept) continue;
    (void)hipStreamSynchronize(c->stream);
    free_graph(c, true);
    st = load_graph(c, n, m, row_ptr, col, w, mem, flags, records);
  }
  if (st == PANTHER_OK) {
    c->err.clear();  // a failed first attempt's message
  } else if (!c->has_graph) {
    // a rejected graph's storage, or the former graph's, serves nothing now
    (void)hipStreamSynchronize(c->stream);
    for (DevBuf panther_ctx::*b : kGraphBuffers) ctx_release(c->*b);
  }
  return st;
}

// ---------------------------------------------------------------------------
// sample_paths (a2 walk + a3 index)
// ---------------------------------------------------------------------------
static int build_index(panther_ctx* c) {
  hipStream_t s = c->stream;
  const int32_t n = c->n;
  const uint64_t R = (uint64_t)c->R;
  int bits_total = 1;
  while (bits_total < 31 && (int64_t(1) << bits_total) < (int64_t)n) ++bits_total;
  const int passes = (bits_total + kRadixPassBits - 1) / kRadixPassBits;
  const int pass_bits = (bits_total + passes - 1) / passes;
  const uint64_t tiles1 = radix_tiles_paths(R, c->T);
  // buffers are sized for the pair count's bound R (T+1), so the passes
  // never wait for the host to learn the count
  const uint64_t nnz_cap = R * (uint64_t)(c->T + 1);
  const uint64_t tiles = radix_tiles_pairs(nnz_cap);
  const uint64_t hist_cap = 256 * std::max<uint64_t>(tiles1, tiles);
  TRY(ctx_ensure(c, c->b_hist, sizeof(uint32_t) * hist_cap, "radix histograms"));
  TRY(ctx_ensure(c, c->b_offs, sizeof(uint64_t) * (hist_cap + 1), "radix offsets"));
  TRY(ctx_ensure(c, c->b_stemp, scan_temp_bytes((int64_t)hist_cap), "scan temp"));
  TRY(ctx_ensure(c, c->b_nnz, 64, "pair count"));
  TRY(ctx_ensure(c, c->b_inv_pid, sizeof(uint32_t) * nnz_cap, "index path ids"));
  TRY(ctx_ensure(c, c->b_inv_ptr, sizeof(uint64_t) * (size_t)(n + 1), "index offsets"));
  TRY(ctx_ensure(c, c->b_keys0, sizeof(uint32_t) * nnz_cap, "radix keys"));
  if (passes > 1) TRY(ctx_ensure(c, c->b_keys1, sizeof(uint32_t) * nnz_cap, "radix keys"));
  if (passes > 1) TRY(ctx_ensure(c, c->b_vtmp, sizeof(uint32_t) * nnz_cap, "radix values"));
  uint32_t* hist = static_cast<uint32_t*>(c->b_hist.p);
  uint64_t* offs = static_cast<uint64_t*>(c->b_offs.p);
  uint64_t* d_nnz = static_cast<uint64_t*>(c->b_nnz.p);
  void* stemp = c->b_stemp.p;
  c->d_inv_pid = static_cast<uint32_t*>(c->b_inv_pid.p);
  c->d_inv_ptr = static_cast<uint64_t*>(c->b_inv_ptr.p);
  uint32_t* keys[2] = {static_cast<uint32_t*>(c->b_keys0.p),
                       static_cast<uint32_t*>(c->b_keys1.p)};
  uint32_t* vtmp = static_cast<uint32_t*>(c->b_vtmp.p);
  // pass p writes its values to inv_pid when (passes - p) is even, so the
  // last pass lands in inv_pid
  auto vals_of = [&](int pass) { return ((passes - pass) % 2 == 0) ? c->d_inv_pid : vtmp; };
  // pass 1: histograms straight from the path rows; the scan's total is
  // the pair count
  int shift = 0;
  int bits = std::min(pass_bits, bits_total - shift);
  launch_radix_up_paths(c->stride, c->d_paths, R, c->T, shift, bits, hist, s);
  launch_scan_u32_to_u64(hist, offs, (int64_t)(256 * tiles1), stemp, s);
  launch_copy_u64(offs + 256 * tiles1, d_nnz, s);
  launch_radix_down_paths(c->stride, c->d_paths, R, c->T, shift, bits, offs, keys[0], vals_of(1),
                          s);
  HIPTRY(hipGetLastError(), "index pass 1");
  for (int pass = 2; pass <= passes; ++pass) {
    shift += bits;
    bits = std::min(pass_bits, bits_total - shift);
    const uint32_t* kin = keys[(pass - 2) % 2];
    uint32_t* kout = keys[(pass - 1) % 2];
    launch_radix_up_pairs(kin, d_nnz, nnz_cap, shift, bits, hist, s);
    launch_scan_u32_to_u64(hist, offs, (int64_t)(256 * tiles), stemp, s);
    launch_radix_down_pairs(kin, vals_of(pass - 1), d_nnz, nnz_cap, shift, bits, offs, kout,
                            vals_of(pass), s);
    HIPTRY(hipGetLastError(), "index pass");
  }
  launch_list_bounds(keys[(passes - 1) % 2], d_nnz, nnz_cap, n, c->d_inv_ptr, s);
  HIPTRY(hipGetLastError(), "index bounds");
  return PANTHER_OK;
}

extern "C" int panther_sample_paths(panther_ctx* c, int32_t T, int64_t R, uint64_t seed) {
  if (!c) return PANTHER_EINVAL;
  c->err.clear();
  if (!c->has_graph) return ctx_fail(c, PANTHER_ESTATE, "sample_paths before load_graph");
  if (T < 1 || T > 63) return ctx_fail(c, PANTHER_EINVAL, "T must lie in [1, 63]");
  if (R < 1 || R >= (int64_t(1) << 32)) return ctx_fail(c, PANTHER_EINVAL, "R must lie in [1, 2^32)");
  if (hipSetDevice(c->device) != hipSuccess) return ctx_fail(c, PANTHER_EDEVICE, "hipSetDevice");
  free_paths(c, false);
  int stride = 4;
  while (stride < T + 1) stride <<= 1;
  c->T = T;
  c->R = R;
  c->seed = seed;
  c->stride = stride;
  void* p;
  int st = ctx_ensure(c, c->b_paths, sizeof(int32_t) * (size_t)R * (size_t)stride, "paths");
  if (st) return st;
  c->d_paths = static_cast<int32_t*>(c->b_paths.p);
  stage_begin(c, 0, c->stream);
  if (c->pfx64)
    launch_walk64(stride, c->d_vrec, c->d_pfx + 1, c->d_col, c->d_fat,
                  c->d_vstart, c->nstart, T, (uint64_t)R, seed, c->d_paths, c->stream);
  else
    launch_walk32(stride, c->d_vrec, c->d_edge, c->d_fat, c->m, c->d_start_rec, c->nstart, T,
                  (uint64_t)R, seed, c->d_paths, c->stream);
  stage_end(c, 0, c->stream);
  st = ctx_hip(c, hipGetLastError(), "walk");
  if (!st) {
    stage_begin(c, 1, c->stream);
    st = build_index(c);
    stage_end(c, 1, c->stream);
  }
  if (!st) {
    uint64_t nnz = 0;
    st = ctx_hip(c, hipMemcpyAsync(&nnz, c->b_nnz.p, 8, hipMemcpyDeviceToHost, c->stream),
                 "pair count");
    if (!st) st = ctx_hip(c, hipStreamSynchronize(c->stream), "pair count");
    c->nnz = (int64_t)nnz;
  }
  if (!st && !c->d_cnt) {
    // dense per-vertex scratch of the query kernels
    st = ctx_alloc(c, &p, sizeof(uint32_t) * (size_t)c->n, "query counters");
    if (!st) {
      c->d_cnt = static_cast<uint32_t*>(p);
      st = ctx_alloc(c, &p, sizeof(int32_t) * (size_t)c->n, "query touched list");
    }
    if (!st) {
      c->d_touched = static_cast<int32_t*>(p);
      st = ctx_alloc(c, &p, 64, "query control");
    }
    if (!st) {
      c->d_ctl = static_cast<uint32_t*>(p);
      st = ctx_hip(c, hipMemsetAsync(c->d_cnt, 0, sizeof(uint32_t) * (size_t)c->n, c->stream),
                   "query scratch");
    }
    if (!st) st = ctx_hip(c, hipMemsetAsync(c->d_ctl, 0, 64, c->stream), "query scratch");
  }
  if (!st) st = ctx_hip(c, hipStreamSynchronize(c->stream), "sample_paths");
  if (st) {
    free_paths(c, true);
    return st;
  }
  c->has_paths = true;
  return PANTHER_OK;
}

// ---------------------------------------------------------------------------
// accessors
// ---------------------------------------------------------------------------
extern "C" int panther_get_paths(panther_ctx* c, int32_t* out, int mem) {
  if (!c) return PANTHER_EINVAL;
  c->err.clear();
  if (!c->has_paths) return ctx_fail(c, PANTHER_ESTATE, "no paths sampled");
  if (!out) return ctx_fail(c, PANTHER_EINVAL, "null output");
  if (hipSetDevice(c->device) != hipSuccess) return ctx_fail(c, PANTHER_EDEVICE, "hipSetDevice");
  const size_t w = sizeof(int32_t) * (size_t)(c->T + 1);
  if (mem == PANTHER_MEM_DEVICE) {
    launch_pack_paths(c->d_paths, c->stride, c->T + 1, c->R, out, c->stream);
    HIPTRY(hipGetLastError(), "get_paths");
  } else {
    // rows are packed on the device chunk by chunk (a strided copy straight
    // to host memory moves one short row at a time), then copied whole
    const size_t chunk = (size_t)1 << 22;  // rows per chunk
    void* p;
    TRY(ctx_alloc(c, &p, w * std::min<size_t>(chunk, (size_t)c->R), "path staging"));
    Temp tmp;
    tmp.add(p);
    for (size_t r0 = 0; r0 < (size_t)c->R; r0 += chunk) {
      const size_t rows = std::min<size_t>(chunk, (size_t)c->R - r0);
      launch_pack_paths(c->d_paths + r0 * (size_t)c->stride, c->stride, c->T + 1, (int64_t)rows,
                        static_cast<int32_t*>(p), c->stream);
      HIPTRY(hipGetLastError(), "get_paths");
      HIPTRY(hipMemcpyAsync(reinterpret_cast<char*>(out) + r0 * w, p, w * rows,
                            hipMemcpyDeviceToHost, c->stream),
             "get_paths");
    }
    HIPTRY(hipStreamSynchronize(c->stream), "get_paths");
    return PANTHER_OK;
  }
  HIPTRY(hipStreamSynchronize(c->stream), "get_paths");
  return PANTHER_OK;
}

extern "C" int64_t panther_index_nnz(const panther_ctx* c) {
  if (!c) return PANTHER_EINVAL;
  if (!c->has_paths) return PANTHER_ESTATE;
  return c->nnz;
}

extern "C" int panther_get_index(panther_ctx* c, int64_t* inv_ptr, uint32_t* inv_pid, int mem) {
  if (!c) return PANTHER_EINVAL;
  c->err.clear();
  if (!c->has_paths) return ctx_fail(c, PANTHER_ESTATE, "no paths sampled");
  if (!inv_ptr || (c->nnz && !inv_pid)) return ctx_fail(c, PANTHER_EINVAL, "null output");
  const hipMemcpyKind kind =
      mem == PANTHER_MEM_DEVICE ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
  HIPTRY(hipMemcpyAsync(inv_ptr, c->d_inv_ptr, sizeof(int64_t) * (size_t)(c->n + 1), kind,
                        c->stream),
         "get_index");
  if (c->nnz)
    HIPTRY(hipMemcpyAsync(inv_pid, c->d_inv_pid, sizeof(uint32_t) * (size_t)c->nnz, kind,
                          c->stream),
           "get_index");
  HIPTRY(hipStreamSynchronize(c->stream), "get_index");
  return PANTHER_OK;
}

// ---------------------------------------------------------------------------
// query validation shared by topk_similar and pp_topk: returns the queries
// on the host (for range checks and the plain form's launch sizes) and on
// the device.
// ---------------------------------------------------------------------------
int stage_queries(panther_ctx* c, const int32_t* queries, int64_t nq, int mem, hipStream_t s,
                  std::vector<int32_t>& hq, const int32_t** dq, void** dq_owned) {
  *dq_owned = nullptr;
  hq.resize((size_t)nq);
  if (mem == PANTHER_MEM_HOST) {
    std::memcpy(hq.data(), queries, sizeof(int32_t) * (size_t)nq);
  } else {
    HIPTRY(hipMemcpyAsync(hq.data(), queries, sizeof(int32_t) * (size_t)nq, hipMemcpyDeviceToHost,
                          s),
           "queries");
    HIPTRY(hipStreamSynchronize(s), "queries");
  }
  for (int64_t i = 0; i < nq; ++i)
    if (hq[i] < 0 || hq[i] >= c->n)
      return ctx_fail(c, PANTHER_ERANGE, "query %lld (= %d) outside [0, %d)", (long long)i, hq[i],
                      c->n);
  if (mem == PANTHER_MEM_DEVICE) {
    *dq = queries;
  } else {
    void* p;
    TRY(ctx_alloc(c, &p, sizeof(int32_t) * (size_t)nq, "queries"));
    *dq_owned = p;
    HIPTRY(hipMemcpyAsync(p, hq.data(), sizeof(int32_t) * (size_t)nq, hipMemcpyHostToDevice, s),
           "queries");
    *dq = static_cast<const int32_t*>(p);
  }
  return PANTHER_OK;
}

void free_lane(Lane* lane) {
  free_batch_state(lane);
  for (DevBuf* b : {&lane->b_qlen, &lane->b_pool, &lane->b_out, &lane->b_stats, &lane->b_q,
                    &lane->b_qrows, &lane->b_fb, &lane->b_fbw, &lane->b_qsort,
                    &lane->b_qsort_tmp, &lane->b_rep, &lane->b_seen})
    ctx_release(*b);
  pinned_release(lane->h_qlen);
  lane->have_stats = false;
}

int query_lengths(panther_ctx* c, Lane* lane, const int32_t* dq, int64_t nq, hipStream_t s,
                  const uint64_t** len, bool to_host, bool once) {
  const size_t bytes = sizeof(uint64_t) * (size_t)std::max<int64_t>(nq, 1);
  TRY(ctx_ensure(c, lane->b_qlen, bytes, "query lengths"));
  uint64_t* qlen = static_cast<uint64_t*>(lane->b_qlen.p);
  // without room for the scratch every query is answered by itself
  once = once && nq > 1 && nq < ((int64_t)1 << 31) &&
         ctx_ensure(c, lane->b_rep, sizeof(int32_t) * (size_t)nq, nullptr) == PANTHER_OK;
  // Marks: a word per vertex, or, for up to 1,024 queries, a hash of 32 words
  // or more per query.  (The hash spares the first call on a graph the clearing
  // of n words; at 10,000 queries and three slots each its longest chains of
  // atomics made every call 4 per cent slower: 0.201 -> 0.208 ms.)
  uint64_t slots = 32;
  while (slots < 32 * (uint64_t)nq) slots <<= 1;
  const bool direct = nq > 1024 || slots >= (uint64_t)c->n;
  const size_t seen_bytes = sizeof(uint64_t) * (size_t)(direct ? (uint64_t)c->n : slots);
  // (after b_rep, whose allocation may have given b_seen back)
  const bool fresh = !lane->b_seen.p || lane->b_seen.cap < seen_bytes || lane->seen_call == ~0u;
  if (once && ctx_ensure(c, lane->b_seen, seen_bytes, nullptr) == PANTHER_OK) {
    if (fresh) {
      lane->seen_call = ~0u;  // not cleared, should the clearing fail
      HIPTRY(hipMemsetAsync(lane->b_seen.p, 0, lane->b_seen.cap, s), "repeated queries");
      lane->seen_call = 0;
    }
    ++lane->seen_call;
    launch_query_lengths_once(c->d_inv_ptr, dq, nq,
                              static_cast<unsigned long long*>(lane->b_seen.p),
                              direct ? ~0u : (uint32_t)(slots - 1), lane->seen_call,
                              static_cast<int32_t*>(lane->b_rep.p), qlen, s);
  } else {
    launch_query_lengths(c->d_inv_ptr, dq, nq, qlen, s);
  }
  HIPTRY(hipGetLastError(), "query lengths");
  if (!to_host) {
    *len = nullptr;
    return PANTHER_OK;
  }
  TRY(pinned_ensure(c, lane->h_qlen, bytes, "query lengths"));
  HIPTRY(hipMemcpyAsync(lane->h_qlen.p, lane->b_qlen.p, sizeof(uint64_t) * (size_t)nq,
                        hipMemcpyDeviceToHost, s),
         "query lengths");
  HIPTRY(hipStreamSynchronize(s), "query lengths");
  *len = static_cast<const uint64_t*>(lane->h_qlen.p);
  return PANTHER_OK;
}

// ---------------------------------------------------------------------------
// all-vertex top-k: the batched form over queries 0..n-1
// ---------------------------------------------------------------------------
extern "C" int panther_topk_all(panther_ctx* c, int32_t k, int32_t* out_ids, uint32_t* out_counts,
                                int32_t* out_len, int mem, void* stream) {
  if (!c) return PANTHER_EINVAL;
  c->err.clear();
  if (!c->has_paths) return ctx_fail(c, PANTHER_ESTATE, "topk_all before sample_paths");
  if (k < 1 || k > 1024) return ctx_fail(c, PANTHER_EINVAL, "k must lie in [1, 1024]");
  if (mem != PANTHER_MEM_HOST && mem != PANTHER_MEM_DEVICE)
    return ctx_fail(c, PANTHER_EINVAL, "bad mem");
  if (!out_ids || !out_counts || !out_len) return ctx_fail(c, PANTHER_EINVAL, "null buffer");
  if (hipSetDevice(c->device) != hipSuccess) return ctx_fail(c, PANTHER_EDEVICE, "hipSetDevice");
  hipStream_t s = pick_stream(c, stream);
  const int64_t n = c->n;
  TRY(ctx_ensure(c, c->b_allv, sizeof(int32_t) * (size_t)n, "vertex ids"));
  int32_t* ids = static_cast<int32_t*>(c->b_allv.p);
  int32_t* d_ids = out_ids;
  uint32_t* d_cnt = out_counts;
  int32_t* d_len = out_len;
  Temp tmp;
  if (mem == PANTHER_MEM_HOST) {
    void* p;
    TRY(ctx_alloc(c, &p, (sizeof(int32_t) + sizeof(uint32_t)) * (size_t)n * (size_t)k +
                             sizeof(int32_t) * (size_t)n,
                  "all-vertex outputs"));
    tmp.add(p);
    d_ids = static_cast<int32_t*>(p);
    d_cnt = reinterpret_cast<uint32_t*>(d_ids + (size_t)n * k);
    d_len = reinterpret_cast<int32_t*>(d_cnt + (size_t)n * k);
  }
  TRY(order_begin(c, s));
  stage_begin(c, 2, s);
  launch_iota(ids, (int32_t)n, s);
  HIPTRY(hipGetLastError(), "vertex ids");
  const uint64_t* qlen = nullptr;
  TRY(query_lengths(c, &c->lane0, ids, n, s, &qlen, !batched_plan_on_device(n)));
  TRY(run_batched(c, &c->lane0, ids, qlen, n, k, d_ids, d_cnt, d_len, nullptr, s));
  stage_end(c, 2, s);
  TRY(order_end(c, s));
  if (mem == PANTHER_MEM_HOST) {
    HIPTRY(hipMemcpyAsync(out_ids, d_ids, sizeof(int32_t) * (size_t)n * k, hipMemcpyDeviceToHost,
                          s),
           "all-vertex outputs");
    HIPTRY(hipMemcpyAsync(out_counts, d_cnt, sizeof(uint32_t) * (size_t)n * k,
                          hipMemcpyDeviceToHost, s),
           "all-vertex outputs");
    HIPTRY(hipMemcpyAsync(out_len, d_len, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost, s),
           "all-vertex outputs");
    HIPTRY(hipStreamSynchronize(s), "topk_all");
  }
  return PANTHER_OK;
}

// ---------------------------------------------------------------------------
// topk_similar (a4 + a5; a8 in the batched form)
// ---------------------------------------------------------------------------
extern "C" int panther_topk_similar(panther_ctx* c, const int32_t* queries, int64_t nq, int32_t k,
                                    int32_t* out_ids, uint32_t* out_counts, int32_t* out_len,
                                    int mem, void* stream) {
  if (!c) return PANTHER_EINVAL;
  c->err.clear();
  if (!c->has_paths) return ctx_fail(c, PANTHER_ESTATE, "topk_similar before sample_paths");
  if (k < 1 || k > 1024) return ctx_fail(c, PANTHER_EINVAL, "k must lie in [1, 1024]");
  if (nq < 0) return ctx_fail(c, PANTHER_EINVAL, "nq must be >= 0");
  if (mem != PANTHER_MEM_HOST && mem != PANTHER_MEM_DEVICE)
    return ctx_fail(c, PANTHER_EINVAL, "bad mem");
  if (nq == 0) return PANTHER_OK;
  if (!queries || !out_ids || !out_counts || !out_len)
    return ctx_fail(c, PANTHER_EINVAL, "null buffer");
  if (hipSetDevice(c->device) != hipSuccess) return ctx_fail(c, PANTHER_EDEVICE, "hipSetDevice");
  hipStream_t s = pick_stream(c, stream);
  std::vector<int32_t> hq;
  const int32_t* dq = nullptr;
  void* owned = nullptr;
  Temp tmp;
  int st = stage_queries(c, queries, nq, mem, s, hq, &dq, &owned);
  if (owned) tmp.add(owned);
  if (st) return st;
  int32_t* d_ids = out_ids;
  uint32_t* d_cnt = out_counts;
  int32_t* d_len = out_len;
  if (mem == PANTHER_MEM_HOST) {
    void* p;
    TRY(ctx_alloc(c, &p, (sizeof(int32_t) + sizeof(uint32_t)) * (size_t)nq * (size_t)k +
                             sizeof(int32_t) * (size_t)nq,
                  "query outputs"));
    tmp.add(p);
    d_ids = static_cast<int32_t*>(p);
    d_cnt = reinterpret_cast<uint32_t*>(d_ids + (size_t)nq * k);
    d_len = reinterpret_cast<int32_t*>(d_cnt + (size_t)nq * k);
  }
  TRY(order_begin(c, s));
  stage_begin(c, 2, s);
  const uint64_t* qlen = nullptr;
  TRY(query_lengths(c, &c->lane0, dq, nq, s, &qlen,
                    c->topk_form == PANTHER_FORM_PLAIN || !batched_plan_on_device(nq),
                    c->topk_form != PANTHER_FORM_PLAIN));
  if (c->topk_form == PANTHER_FORM_PLAIN) {
    TopkScratch sc{c->d_cnt, c->d_touched, c->d_ctl};
    for (int64_t i = 0; i < nq; ++i) {
      launch_topk_plain(c->stride, dq + i, c->n, c->d_inv_ptr, c->d_inv_pid, c->d_paths, qlen[i],
                        sc, k, d_ids + i * k, d_cnt + i * k, d_len + i, s);
    }
    HIPTRY(hipGetLastError(), "topk plain");
  } else {
    TRY(run_batched(c, &c->lane0, dq, qlen, nq, k, d_ids, d_cnt, d_len, nullptr, s));
  }
  stage_end(c, 2, s);
  TRY(order_end(c, s));
  if (mem == PANTHER_MEM_HOST) {
    HIPTRY(hipMemcpyAsync(out_ids, d_ids, sizeof(int32_t) * (size_t)nq * k, hipMemcpyDeviceToHost,
                          s),
           "topk outputs");
    HIPTRY(hipMemcpyAsync(out_counts, d_cnt, sizeof(uint32_t) * (size_t)nq * k,
                          hipMemcpyDeviceToHost, s),
           "topk outputs");
    HIPTRY(hipMemcpyAsync(out_len, d_len, sizeof(int32_t) * (size_t)nq, hipMemcpyDeviceToHost, s),
           "topk outputs");
    HIPTRY(hipStreamSynchronize(s), "topk");
  } else if (owned) {
    // the staged query copy is freed on return; make sure it is consumed
    HIPTRY(hipStreamSynchronize(s), "topk");
  }
  return PANTHER_OK;
}
