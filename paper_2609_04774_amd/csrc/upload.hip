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
//
// A launch that is being captured into a graph has no such moment: each replay
// reads the source again.  Its tables travel as kernel arguments, which the
// graph keeps for itself, in pieces of the argument space: a node of 1 to 2 us
// each (29 KB, 300 rows of 512 heads: 62 us a replay, 51 a call; 25 KB, the 32K
// shard: 1795 and 1789).
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstring>

#include "internal.h"

namespace cpattn {

namespace {

__global__ __launch_bounds__(256) void upload_tables_kernel(uint4* __restrict__ dst, const uint4* __restrict__ src,
                                                            size_t n16, uint32_t* done) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n16) dst[i] = src[i];
  __syncthreads();  // every load of the block has returned (its stores wait for them)
  if (threadIdx.x == 0) __hip_atomic_store(done + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
static_assert(kUploadBlockBytes == 256 * sizeof(uint4), "one 16-byte piece per thread");

// One piece of the tables among the kernel's arguments, read through the
// argument segment's own address (as InlineTables are).
struct ChunkArgs {
  uint4* dst;
  int n16;
  InlineTables chunk;
};

__global__ __launch_bounds__(256) void upload_chunk_kernel(uint4* __restrict__ dst, int n16, InlineTables) {
  typedef const __attribute__((address_space(4))) unsigned char* Args;
  const Args src = (Args)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(ChunkArgs, chunk);
  if ((int)threadIdx.x < n16) dst[threadIdx.x] = ((const uint4*)(src))[threadIdx.x];
}
static_assert(kInlineBytes % sizeof(uint4) == 0 && kInlineBytes <= 256 * sizeof(uint4), "one 16-byte piece per thread");

int launched() {
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? CP_OK : fail(CP_ERR_HIP, std::string("table upload launch: ") + hipGetErrorString(e));
}

}  // namespace

int launch_upload(void* dst, const void* src, size_t bytes, void* stream) {
  if (bytes == 0) return CP_OK;
  if (bytes % 16 || (uintptr_t)dst % 16 || (uintptr_t)src % 16)
    return fail(CP_ERR_INVALID, "table upload: sizes and addresses must be multiples of 16 bytes");
  if (!capturing(stream)) {
    uint32_t* done = reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(const_cast<void*>(src)) + bytes);
    hipLaunchKernelGGL(upload_tables_kernel, dim3((unsigned)upload_blocks(bytes)), dim3(256), 0, (hipStream_t)stream,
                       static_cast<uint4*>(dst), static_cast<const uint4*>(src), bytes / 16, done);
    return launched();
  }
  InlineTables chunk;
  int st = CP_OK;
  for (size_t at = 0; st == CP_OK && at < bytes; at += kInlineBytes) {
    const size_t n = bytes - at < kInlineBytes ? bytes - at : kInlineBytes;
    std::memcpy(chunk.bytes, static_cast<const unsigned char*>(src) + at, n);
    hipLaunchKernelGGL(upload_chunk_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream,
                       reinterpret_cast<uint4*>(static_cast<unsigned char*>(dst) + at), (int)(n / 16), chunk);
    st = launched();
  }
  return st;
}

}  // namespace cpattn
