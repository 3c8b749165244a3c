// Host-only check of how a launch's tables reach the workspace
// (tests/test_tables.py builds and runs it; no GPU is touched): the runtime
// calls of the staging code are replaced by the functions below.
//   * A captured launch takes no staging slot: its graph runs the upload again
//     after the slots have other uses.
// Prints "ok" on success, else the first failure, and exits non-zero.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <vector>

namespace fake {
bool capturing = false;
std::vector<std::pair<unsigned char*, size_t>> pinned;  // live allocations
hipError_t is_capturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t host_malloc(void** p, size_t n, unsigned) {
  *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
  pinned.push_back({static_cast<unsigned char*>(*p), n});
  return hipSuccess;
}
hipError_t host_free(void* p) {
  for (size_t i = 0; i < pinned.size(); ++i)
    if (pinned[i].first == p) pinned.erase(pinned.begin() + i);
  std::free(p);
  return hipSuccess;
}
hipError_t device_pointer(void** d, void* p, unsigned) {
  *d = p;
  return hipSuccess;
}
bool is_pinned(const void* p) {
  for (const auto& x : pinned)
    if (p >= x.first && p < x.first + x.second) return true;
  return false;
}
}  // namespace fake
#define hipStreamIsCapturing fake::is_capturing
#define hipHostMalloc fake::host_malloc
#define hipHostFree fake::host_free
#define hipHostGetDevicePointer fake::device_pointer

#include "../paper_2609_04774_amd/csrc/cp_attn.cpp"

namespace {

int failures = 0;
int uploads = 0, uploads_from_slots = 0;

void expect(bool ok, const char* what) {
  if (!ok && failures++ == 0) std::printf("FAIL %s\n", what);
}

}  // namespace

namespace cpattn {
int launch_partial(const PartialParams&, void*) { return CP_OK; }
int launch_merge(const MergeParams&, void*) { return 1; }
// Copies as the kernel would; the words after a slot's tables are set.
int launch_upload(void* dst, const void* src, size_t bytes, void*) {
  ++uploads;
  std::memcpy(dst, src, bytes);
  if (!fake::is_pinned(src)) return CP_OK;
  ++uploads_from_slots;
  uint32_t* done = reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(const_cast<void*>(src)) + bytes);
  for (size_t i = 0; i < upload_blocks(bytes); ++i) done[i] = 1;
  return CP_OK;
}
}  // namespace cpattn

namespace {

// One cp_attn_partial of `heads` heads (tables beyond the argument space) into
// a workspace in host memory, whose tables are compared with the plan's.
void launch(int heads, const char* what) {
  cp_partial_desc d;
  std::memset(&d, 0, sizeof(d));
  make_plan(0, 200, 1, 0, &d.plan);
  void* f = reinterpret_cast<void*>(0x100000);
  d.q = d.k_new = d.v_new = f;
  d.o = d.lse = static_cast<float*>(f);
  d.kv_rank = CP_KV_ALL;
  Plan plan;
  expect(build_plan(&d, 1, heads, heads, kTargetPieces, &plan) == CP_OK, "build_plan");
  const Layout lay = layout_of(plan);
  InlineTables inl;
  expect(!pack_inline(plan, &inl), "the tables fit the argument space");
  void* ws = std::aligned_alloc(256, (lay.total + 255) / 256 * 256);
  expect(cp_attn_partial(&d, 1, heads, heads, 128, 0.f, ws, lay.total, nullptr) == CP_OK, what);
  expect(std::memcmp(static_cast<unsigned char*>(ws) + lay.items, plan.items.data(),
                     plan.items.size() * sizeof(WorkItem)) == 0, what);
  std::free(ws);
}

}  // namespace

int main() {
  for (int i = 0; i < 20; ++i) launch(425 + 97 * (7 * i % 20), "staged launch");
  expect(uploads == 20 && uploads_from_slots == 20, "staged launches upload from slots");
  fake::capturing = true;
  for (int i = 0; i < 20; ++i) launch(425 + 97 * (7 * i % 20), "captured launch");
  expect(uploads == 40 && uploads_from_slots == 20, "a captured launch uploads from a slot");
  if (failures) return 1;
  std::printf("ok\n");
  return 0;
}
