// Small device tables owned by a plan (chirps and filter spectra of the 1-D
// transforms, roots of unity of the filter DFT, inverse-DFT weights of the
// weight gradient, operands of the matrix-product transforms).  Each is built
// in double precision, on the host and uploaded or by a kernel, in the plan's
// first call that needs it on a device; the plan frees them when it is destroyed.
#include <cstring>
#include <functional>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "common.hpp"

namespace blc {
namespace {

struct TabEntry {
  int dev;
  std::vector<long> key;
  float2* d;
  const TableScope* making;  // the call whose kernel makes it, until that has been waited for
};
// Small tables share allocations: a plan's first calls make up to five, and an
// allocation costs about 5 us (first training step, 32 x 25 points 192 -> 177 us).
constexpr size_t kChunk = 512 * 1024, kSmallTable = kChunk / 2;  // bytes
struct Chunk {
  int dev;
  char* d;
  size_t used;
};
struct PlanTables {
  std::vector<TabEntry> entries;
  std::vector<Chunk> chunks;
  std::vector<std::pair<int, float2*>> large;  // (device, allocation) of the others
};
std::mutex g_tab_mu;
thread_local TableScope* t_scope = nullptr;

bool capturing(hipStream_t s) {
  hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &c) != hipSuccess) (void)hipGetLastError();
  return c != hipStreamCaptureStatusNone;
}

// The table of `key` on the current device, made by `make` (which allocates
// and fills it) where the plan has none yet.
bl_status_t find_or_make(const bl_conv_plan_s* p, const std::vector<long>& key, hipStream_t s, const float2** out,
                         const std::function<bl_status_t(PlanTables&, int, float2**)>& make) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return BL_ERR_HIP;
  std::lock_guard<std::mutex> lk(g_tab_mu);
  if (!p->tables) p->tables = new (std::nothrow) PlanTables();
  auto* cache = static_cast<PlanTables*>(p->tables);
  if (!cache) return BL_ERR_OOM;
  for (const TabEntry& e : cache->entries)
    if (e.dev == dev && e.key == key) {
      if (e.making && e.making != t_scope) {  // (under the lock: the scope is still there)
        if (capturing(s)) return BL_ERR_UNSUPPORTED;
        if (hipEventSynchronize(e.making->made) != hipSuccess) return BL_ERR_HIP;
      }
      *out = e.d;
      return BL_OK;
    }
  // a stream that is being captured allows no allocation and no wait: the
  // caller takes a path without the table, if it has one
  if (capturing(s)) return BL_ERR_UNSUPPORTED;
  float2* d = nullptr;
  const bl_status_t st = make(*cache, dev, &d);
  if (st != BL_OK) return st;  // (what it allocated goes with the plan)
  const bool waits = t_scope && t_scope->pending;  // for a kernel of this call
  if (waits) t_scope->cache = cache, t_scope->pending = false;
  cache->entries.push_back(TabEntry{dev, key, d, waits ? t_scope : nullptr});
  *out = d;
  return BL_OK;
}

// Memory for a table of n float2 on the current device dev.
bl_status_t allocate(PlanTables& t, int dev, size_t n, float2** d) {
  const size_t bytes = (n * sizeof(float2) + 255) / 256 * 256;
  const bool small = bytes <= kSmallTable;
  if (small)
    for (Chunk& c : t.chunks)
      if (c.dev == dev && c.used + bytes <= kChunk) {
        *d = reinterpret_cast<float2*>(c.d + c.used);
        c.used += bytes;
        return BL_OK;
      }
  void* m = nullptr;
  if (hipMalloc(&m, small ? kChunk : bytes) != hipSuccess) {
    (void)hipGetLastError();
    return BL_ERR_OOM;
  }
  *d = static_cast<float2*>(m);
  if (small)
    t.chunks.push_back(Chunk{dev, static_cast<char*>(m), bytes});
  else
    t.large.emplace_back(dev, *d);
  return BL_OK;
}

}  // namespace

bl_status_t plan_table(const bl_conv_plan_s* p, const std::vector<long>& key,
                       const std::function<void(std::vector<float2>&)>& build, const float2** out, hipStream_t s) {
  return find_or_make(p, key, s, out, [&](PlanTables& t, int dev, float2** d) {
    std::vector<float2> host;
    build(host);
    const bl_status_t st = allocate(t, dev, host.size(), d);
    if (st != BL_OK) return st;
    return hipMemcpy(*d, host.data(), host.size() * sizeof(float2), hipMemcpyHostToDevice) == hipSuccess ? BL_OK
                                                                                                        : BL_ERR_HIP;
  });
}

bl_status_t plan_table_on_device(const bl_conv_plan_s* p, const std::vector<long>& key, size_t n,
                                 const std::function<void(float2*)>& fill, const float2** out, hipStream_t s) {
  return find_or_make(p, key, s, out, [&](PlanTables& held, int dev, float2** d) {
    const bl_status_t st = allocate(held, dev, n, d);
    if (st != BL_OK) return st;
    fill(*d);
    if (hipGetLastError() != hipSuccess) return BL_ERR_HIP;
    // waited for: a call on another stream may be the next to read it
    if (TableScope* t = t_scope) {
      if (!t->made && hipEventCreateWithFlags(&t->made, hipEventDisableTiming) != hipSuccess) t->made = nullptr;
      if (t->made && hipEventRecord(t->made, s) == hipSuccess) {
        t->pending = true;
        return BL_OK;
      }
      (void)hipGetLastError();
    }
    return hipStreamSynchronize(s) == hipSuccess ? BL_OK : BL_ERR_HIP;
  });
}

TableScope::TableScope() { t_scope = this; }

TableScope::~TableScope() {
  t_scope = nullptr;
  if (!made) return;
  (void)hipEventSynchronize(made);
  std::lock_guard<std::mutex> lk(g_tab_mu);
  if (cache)
    for (TabEntry& e : static_cast<PlanTables*>(cache)->entries)
      if (e.making == this) e.making = nullptr;
  (void)hipEventDestroy(made);
}

bl_status_t lds_opt_in(const void* kern, int bytes) {
  static std::mutex mu;
  static std::vector<std::pair<const void*, int>> done;  // (kernel, device)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return BL_ERR_HIP;
  std::lock_guard<std::mutex> lk(mu);
  for (const auto& e : done)
    if (e.first == kern && e.second == dev) return BL_OK;
  if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) return BL_ERR_HIP;
  done.emplace_back(kern, dev);
  return BL_OK;
}

int device_cus() {
  static int count[64];  // per device; written once with the same value
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (count[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    count[dev] = n;
  }
  return count[dev];
}

long float_key(float x) {
  unsigned u;
  std::memcpy(&u, &x, sizeof u);
  return (long)u;
}

}  // namespace blc

void bl_plan_tables_free(void* tables) {
  if (!tables) return;
  auto* c = static_cast<blc::PlanTables*>(tables);
  int cur = 0;
  const bool have = hipGetDevice(&cur) == hipSuccess;
  for (const auto& e : c->large)
    if (hipSetDevice(e.first) == hipSuccess) (void)hipFree(e.second);
  for (const blc::Chunk& e : c->chunks)
    if (hipSetDevice(e.dev) == hipSuccess) (void)hipFree(e.d);
  if (have) (void)hipSetDevice(cur);
  delete c;
}
