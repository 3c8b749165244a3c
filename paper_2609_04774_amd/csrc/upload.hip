// The launch tables' upload.  Each cp_attn_partial call copies its
// descriptors, work list and split list (a few KB to a few hundred KB) from
// the library's pinned host staging into the caller's workspace.  A copy
// engine transfer (hipMemcpyAsync) makes the compute queue wait for the copy
// engine's completion signal before the attention kernel starts, about 17 us
// per call on this GPU; a kernel on the same stream reads the staging over
// the bus instead and hands over like any two kernels do (about 7 us in
// all).  16 bytes per thread.
//
// A staging slot may be written again once the kernel has read it.  Each block
// says so itself, in a word after the source: an event recorded behind the
// kernel holds the attention kernel back until the queue has signalled it
// (5.6 us between the two kernels of every call).
#include <hip/hip_runtime.h>

#include "internal.h"

namespace cpattn {

namespace {

__global__ __launch_bounds__(256) void upload_tables_kernel(uint4* __restrict__ dst, const uint4* __restrict__ src,
                                                            size_t n16, uint32_t* done) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n16) dst[i] = src[i];
  __syncthreads();  // every load of the block has returned (its stores wait for them)
  if (done && threadIdx.x == 0) __hip_atomic_store(done + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
static_assert(kUploadBlockBytes == 256 * sizeof(uint4), "one 16-byte piece per thread");

}  // namespace

int launch_upload(void* dst, const void* src, size_t bytes, void* stream) {
  if (bytes == 0) return CP_OK;
  if (bytes % 16 || (uintptr_t)dst % 16 || (uintptr_t)src % 16)
    return fail(CP_ERR_INVALID, "table upload: sizes and addresses must be multiples of 16 bytes");
  const size_t n16 = bytes / 16;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing((hipStream_t)stream, &capture) != hipSuccess) {
    (void)hipGetLastError();
    capture = hipStreamCaptureStatusNone;
  }
  uint32_t* done = nullptr;
  if (capture == hipStreamCaptureStatusNone)
    done = reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(const_cast<void*>(src)) + bytes);
  hipLaunchKernelGGL(upload_tables_kernel, dim3((unsigned)upload_blocks(bytes)), dim3(256), 0, (hipStream_t)stream,
                     static_cast<uint4*>(dst), static_cast<const uint4*>(src), n16, done);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(CP_ERR_HIP, std::string("table upload launch: ") + hipGetErrorString(e));
  return CP_OK;
}

}  // namespace cpattn
