// Host-only check of how a launch's tables reach the workspace
// (tests/test_tables.py builds and runs it; no GPU is touched): the runtime
// calls of the staging code are replaced by the functions below.
//   * A captured launch takes no staging slot: its graph runs the upload again
//     after the slots have other uses.
//   * A launch whose slot is still being read waits for that upload alone, for
//     as long as the runtime says that its stream has work: it never waits for
//     the device, asks on the upload's device and in relaxed capture mode, and
//     launches from other slots meanwhile.  An upload that will not run is an
//     error, once.
// Prints "ok" on success, else the first failure, and exits non-zero.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <functional>
#include <thread>
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
// A stream's state, what was asked of it and how.
hipError_t stream_state = hipSuccess;
int device = 0, device_syncs = 0, asked = 0, asked_elsewhere = 0, asked_strictly = 0;
hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
std::function<void()> when_asked;
hipError_t device_sync() {
  ++device_syncs;
  return hipErrorUnknown;
}
hipError_t get_device(int* d) {
  *d = device;
  return hipSuccess;
}
hipError_t set_device(int d) {
  device = d;
  return hipSuccess;
}
hipError_t exchange_mode(hipStreamCaptureMode* m) {
  std::swap(*m, mode);
  return hipSuccess;
}
hipError_t stream_query(hipStream_t) {
  ++asked;
  asked_elsewhere += device != 1;
  asked_strictly += mode != hipStreamCaptureModeRelaxed;
  if (when_asked) when_asked();
  return stream_state;
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
#define hipDeviceSynchronize fake::device_sync
#define hipGetDevice fake::get_device
#define hipSetDevice fake::set_device
#define hipThreadExchangeStreamCaptureMode fake::exchange_mode
#define hipStreamQuery fake::stream_query

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
// Copies as the kernel would; the words after a slot's tables are set, at once
// or (stalled) by run_stalled().
bool stalled = false;
std::vector<std::pair<uint32_t*, size_t>> pending;
void run_stalled() {
  for (const auto& p : pending)
    for (size_t i = 0; i < p.second; ++i) __atomic_store_n(p.first + i, 1u, __ATOMIC_RELEASE);
  pending.clear();
}
int launch_upload(void* dst, const void* src, size_t bytes, void*) {
  ++uploads;
  std::memcpy(dst, src, bytes);
  if (!fake::is_pinned(src)) return CP_OK;
  ++uploads_from_slots;
  uint32_t* done = reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(const_cast<void*>(src)) + bytes);
  pending.push_back({done, upload_blocks(bytes)});
  if (!stalled) run_stalled();
  return CP_OK;
}
}  // namespace cpattn

namespace {

// One cp_attn_partial of `heads` heads (tables beyond the argument space) into
// a workspace in host memory, whose tables are compared with the plan's.
int launch(int heads, const char* what, int expected = CP_OK) {
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
  const int st = cp_attn_partial(&d, 1, heads, heads, 128, 0.f, ws, lay.total, nullptr);
  expect(st == expected, what);
  if (st == CP_OK)
    expect(std::memcmp(static_cast<unsigned char*>(ws) + lay.items, plan.items.data(),
                       plan.items.size() * sizeof(WorkItem)) == 0, what);
  std::free(ws);
  return st;
}

}  // namespace

int main() {
  for (int i = 0; i < 20; ++i) launch(425 + 97 * (7 * i % 20), "staged launch");
  expect(uploads == 20 && uploads_from_slots == 20, "staged launches upload from slots");
  fake::capturing = true;
  for (int i = 0; i < 20; ++i) launch(425 + 97 * (7 * i % 20), "captured launch");
  expect(uploads == 40 && uploads_from_slots == 20, "a captured launch uploads from a slot");
  fake::capturing = false;

  // Device 1's uploads stall; a launch on device 0 needs the first slot again.
  fake::device = 1;
  stalled = true;
  for (int i = 0; i < kSlots; ++i) launch(500, "a launch into a free slot");
  fake::device = 0;
  fake::stream_state = hipErrorNotReady;
  fake::when_asked = [] {
    if (fake::asked == 2) run_stalled();
  };
  launch(500, "a launch that waits");
  expect(fake::asked == 2 && fake::asked_elsewhere == 0 && fake::asked_strictly == 0, "how the stream is asked");
  expect(fake::device == 0 && fake::mode == hipStreamCaptureModeGlobal, "device and mode are put back");
  expect(fake::device_syncs == 0, "the wait is on the whole device");

  // A launch waits for its slot while others pass through theirs.
  run_stalled();
  fake::asked = 0;
  fake::device = 1;
  for (int i = 0; i < kSlots; ++i) launch(500, "a launch into a free slot");
  std::pair<uint32_t*, size_t> first = pending.front();
  pending.erase(pending.begin());
  run_stalled();
  stalled = false;
  bool others_done = false, others_were_done = false;
  fake::when_asked = [&] {
    others_were_done = __atomic_load_n(&others_done, __ATOMIC_ACQUIRE);
    pending.push_back(first);
    run_stalled();
  };
  std::thread waiter([] { launch(500, "a launch that waits"); });
  std::this_thread::sleep_for(std::chrono::milliseconds(500));
  for (int i = 0; i < kSlots - 1; ++i) launch(500, "a launch beside one that waits");
  __atomic_store_n(&others_done, true, __ATOMIC_RELEASE);
  waiter.join();
  expect(others_were_done, "launches with free slots wait for one without");

  // A device that is lost: an error for the launch that needs the slot, and the
  // memory is not used again.
  stalled = true;
  for (int i = 0; i < kSlots; ++i) launch(500, "a launch into a free slot");
  fake::when_asked = nullptr;
  fake::stream_state = hipErrorLaunchFailure;
  launch(500, "an upload that never ran", CP_ERR_HIP);
  const size_t left = fake::pinned.size();
  pending.erase(pending.begin());
  run_stalled();
  for (int i = 0; i < kSlots; ++i) launch(500, "a launch after the error");
  run_stalled();
  expect(fake::pinned.size() == left + 1, "the lost upload's memory is left alone");
  if (failures) return 1;
  std::printf("ok\n");
  return 0;
}
