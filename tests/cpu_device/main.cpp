// One step of calls through the C ABI on the CPU. argv[1]: a file of little-endian int32 words,
// the request header (below), then arrays; argv[2]: where the answer goes.
#include "hip/hip_runtime.h"
#undef asm
#undef volatile
#include <sys/mman.h>

#include "pkv_internal.h"

namespace {

enum Route { kPlanDecode, kNoalloc, kFused, kSeparate, kRect, kBuckets };
struct Request {
  int32_t route, order, compute_units, calls;
  int32_t B, hq, hkv, num_pages, max_pages, max_tasks, S, n_rows, bucket_tokens;
  int32_t given_tasks;  // -1: the plan's list; else that many given records, split_offsets and the count
  int32_t num_tasks;
  float sm_scale;
  pkv_plan_params params;
};

// Memory that ends at an unmapped page (and starts after one), so that an access past it ends the
// program. Rounded up to 16 bytes at the front.
char* guarded(size_t bytes) {
  const size_t page = 4096, n = (bytes + page - 1) / page * page;
  char* m = (char*)mmap(nullptr, n + 2 * page, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
  if (m == MAP_FAILED || mprotect(m + page, n, PROT_READ | PROT_WRITE) != 0) std::abort();
  return m + page + (n - (bytes + 15) / 16 * 16);
}
template <typename T>
T* read(FILE* f, size_t count) {
  T* p = (T*)guarded(count * sizeof(T));
  if (std::fread(p, sizeof(T), count, f) != count) std::abort();
  return p;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc != 3) return 2;
  FILE* f = std::fopen(argv[1], "rb");
  Request r;
  if (!f || std::fread(&r, sizeof(r), 1, f) != 1) return 2;
  emu::order = (unsigned)r.order;
  emu::compute_units = r.compute_units;
  const size_t pool = (size_t)r.num_pages * 16 * r.hkv * 128, qn = (size_t)r.B * r.hq * 128;
  uint16_t *q = read<uint16_t>(f, qn), *k = read<uint16_t>(f, pool), *v = read<uint16_t>(f, pool);
  int32_t *table = read<int32_t>(f, (size_t)r.B * r.max_pages), *lens = read<int32_t>(f, (size_t)r.calls * r.B);
  int32_t* row_ids = r.n_rows > 0 ? read<int32_t>(f, r.n_rows) : nullptr;
  pkv_task* tasks = (pkv_task*)guarded(sizeof(pkv_task) * r.max_tasks);
  int32_t *offsets = (int32_t*)guarded(4 * (r.B + 1)), *count = (int32_t*)guarded(4);
  std::memset(tasks, 0, sizeof(pkv_task) * r.max_tasks);
  if (r.given_tasks >= 0) {
    if (std::fread(tasks, sizeof(pkv_task), r.given_tasks, f) != (size_t)r.given_tasks ||
        std::fread(offsets, 4, r.B + 1, f) != (size_t)r.B + 1)
      return 2;
    *count = r.num_tasks;
  }
  const size_t ws_bytes = pkv_workspace_size(r.B, r.hq, r.hkv, 128, r.max_tasks);
  char* ws = guarded(ws_bytes);
  std::memset(ws, 0xFF, ws_bytes);
  uint16_t* out = (uint16_t*)guarded(2 * qn);
  uint32_t* err = (uint32_t*)guarded(4);
  *err = 0;
  FILE* g = std::fopen(argv[2], "wb");
  if (!g || pkv_workspace_init(ws, ws_bytes, r.B, r.hkv, nullptr) != PKV_OK) return 2;
  for (int c = 0; c < r.calls; ++c) {
    const int32_t* n = lens + (size_t)c * r.B;
    std::memset(out, 0xFF, 2 * qn);
    emu::launches.clear();
    int st = PKV_OK;
    if (r.route == kPlanDecode) {
      st = pkv_plan_decode(q, k, v, r.num_pages, table, r.max_pages, n, r.B, r.hq, r.hkv, 128, &r.params, tasks, r.max_tasks,
                           offsets, count, r.sm_scale, out, ws, ws_bytes, nullptr);
    } else if (r.route == kNoalloc) {
      st = pkv_plan_decode_noalloc(q, k, v, r.num_pages, table, r.max_pages, n, r.B, r.hq, r.hkv, 128, &r.params, tasks,
                                   r.max_tasks, offsets, count, r.sm_scale, out, err, nullptr);
    } else if (r.route == kRect) {
      st = pkv_decode_rect(q, k, v, r.num_pages, table, r.max_pages, n, r.B, r.hq, r.hkv, 128, row_ids, r.n_rows, r.S,
                           r.params.tile_tokens, r.sm_scale, out, ws, ws_bytes, nullptr);
    } else if (r.route == kBuckets) {
      st = pkv_decode_buckets(q, k, v, r.num_pages, table, r.max_pages, n, n, r.B, r.hq, r.hkv, 128, r.bucket_tokens,
                              &r.params, r.sm_scale, out, ws, ws_bytes, nullptr, nullptr);
    } else {
      if (r.given_tasks < 0)
        st = pkv_plan(n, nullptr, r.B, r.max_pages, r.num_pages, &r.params, tasks, r.max_tasks, offsets, count, ws,
                      ws_bytes, nullptr);
      if (st == PKV_OK)
        st = pkv_decode(q, k, v, r.num_pages, table, r.max_pages, n, r.B, r.hq, r.hkv, 128, tasks, offsets, count,
                        r.max_tasks, r.sm_scale, r.route == kFused ? PKV_FUSED_MERGE : 0, out, ws, ws_bytes, nullptr);
    }
    uint32_t bits = 0;
    int32_t left = 0;  // completion counters that are not zero
    for (int i = 0; i < r.B * r.hkv; ++i) left += reinterpret_cast<int32_t*>(ws + pkv::kWsHeaderBytes)[i] != 0;
    pkv_check_device_status(ws, nullptr, &bits);
    int32_t head[4] = {st, (int32_t)(bits | *err), left, *count};
    std::fwrite(head, 4, 4, g);
    std::fwrite(out, 2, qn, g);
    std::fwrite(offsets, 4, r.B + 1, g);
    std::fwrite(tasks, sizeof(pkv_task), r.max_tasks, g);
    if (c == 0)
      for (const auto& l : emu::launches) std::printf("%llx %u\n", (unsigned long long)(uintptr_t)l.first, l.second);
  }
  return std::fclose(g) == 0 ? 0 : 2;
}
