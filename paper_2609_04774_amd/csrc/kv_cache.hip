// KV-cache steps around the attention, all pure row copies (HBM-bound):
//
//  * Paged write-back (paper Sec. 2.2, 7.1, 8): a CP rank's new K/V rows go
//    to their token positions in the block-16 paged cache, position p at
//    physical block block_table[p / 16], slot p % 16.
//  * Re-sharding between CP degrees (Sec. 6.2, 7.2): each row of a
//    destination rank is fetched from the source rank that holds the same
//    global position under the source degree.
//  * Paged gather (Sec. 2.2, 7.1, 7.2): positions of a request read back out
//    of the paged cache into contiguous rows.
//
// A row (of K and of V, where both move alike) is copied by 16, 32 or 64 lanes,
// the fewest that hold a narrow row's 16-byte pieces one each, with up to four
// pieces per lane and tensor loaded before any is stored, so that a row's bytes
// are read and written in fully coalesced accesses and no lane idles on the
// rows of one or two KV heads (256 and 512 bytes).  Row indices are derived in
// closed form from the zigzag plans; no index table is read except the block
// table.
//
// Bound by HBM.  Against one wave per row, K's row before V's: 65536 rows of
// one KV head gathered 20.2 -> 12.0 us, of two 25.2 -> 22.9, re-sharded 28.7 ->
// 20.7; a 128K request of eight re-sharded (two tensors at once) 180 -> 170 us
// (6.3 TB/s).
//
// Stores carry non-temporal hints, and so do the gather's loads (a cached prefix
// is seldom in a cache: 69 us for 48K tokens, 73 with plain loads), while the
// write-back and the re-shard load plainly up to the size of the 256 MB Infinity
// Cache, which may hold the rows their caller has just computed or moved: a
// rank's 16384 rows of the 128K prompt take 20.7 us (6.5 TB/s) whether a cache
// holds them or not, with streaming loads 24-27, and with plain stores 28 when
// none does; a 32K request re-sharded 39 us when one does and 46 when not, with
// streaming loads 44 both ways; one rank's 65536 rows re-sharded 38.5 and 45.6,
// with streaming loads 42.3 and 43.9.  Beyond that size streaming loads are the
// faster: 131000 rows written back 200 against 206 us.
#include <hip/hip_runtime.h>

#include "internal.h"

namespace cpattn {

namespace {

constexpr int kThreads = 256;
constexpr int64_t kInfinityCacheBytes = 256 << 20;
constexpr int kPieces = 4;  // 16-byte pieces of a row and tensor in flight per lane

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// kLanes lanes copy one row of kSets tensors: lane l moves 16-byte pieces l,
// l + kLanes, ...  A null source writes zeros.
// kStream: loads with the non-temporal hint.
template <int kLanes, int kSets, bool kStream>
__device__ __forceinline__ void copy_rows(const unsigned char* const (&src)[kSets], unsigned char* const (&dst)[kSets],
                                          int64_t row_bytes, int lane) {
  const int64_t n = row_bytes >> 4;
  for (int64_t base = 0; base < n; base += kPieces * kLanes) {
    u32x4 v[kPieces][kSets];
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
      const int64_t i = base + lane + kLanes * k;
#pragma unroll
      for (int s = 0; s < kSets; ++s) {
        v[k][s] = u32x4{0u, 0u, 0u, 0u};
        if (i >= n || !src[s]) continue;
        const u32x4* from = reinterpret_cast<const u32x4*>(src[s]) + i;
        v[k][s] = kStream ? __builtin_nontemporal_load(from) : *from;
      }
    }
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
      const int64_t i = base + lane + kLanes * k;
#pragma unroll
      for (int s = 0; s < kSets; ++s)
        if (i < n) __builtin_nontemporal_store(v[k][s], reinterpret_cast<u32x4*>(dst[s]) + i);
    }
  }
}

// This thread's row of the launch.
template <int kLanes>
__device__ __forceinline__ int64_t row_index() {
  return (int64_t)blockIdx.x * (kThreads / kLanes) + threadIdx.x / kLanes;
}

// Global position of a rank's local row t: chunk 0's rows, then chunk 1's.
__device__ __forceinline__ int64_t row_position(const int64_t (&q_begin)[2], const int64_t (&q_len)[2], int64_t t) {
  return t < q_len[0] ? q_begin[0] + t : q_begin[1] + (t - q_len[0]);
}

template <int kLanes, bool kStream>
__global__ __launch_bounds__(kThreads) void kv_writeback_kernel(WritebackParams p) {
  const int64_t t = row_index<kLanes>();
  if (t >= p.n_rows) return;
  const int64_t pos = row_position(p.q_begin, p.q_len, t);
  const int64_t blk = p.block_table[pos / kBlockTokens];
  if (blk < 0 || blk >= p.n_blocks) return;  // outside the cache: nothing is written
  const int64_t dst = (blk * kBlockTokens + pos % kBlockTokens) * p.row_bytes;
  copy_rows<kLanes, 2, kStream>({p.k_rows + t * p.row_bytes, p.v_rows + t * p.row_bytes},
                                {p.k_cache + dst, p.v_cache + dst}, p.row_bytes, threadIdx.x % kLanes);
}

// Where suffix index i sits at degree C with chunk length s: the rank holding
// its chunk c (rank c or 2C-1-c) and the local row there (after that rank's
// first chunk when c is its second).
struct RankRow {
  int64_t rank, row;
};

__device__ __forceinline__ RankRow rank_row(int64_t i, int64_t C, int64_t s, int64_t R) {
  const int64_t c = i / s;
  const int64_t r = c < C ? c : 2 * C - 1 - c;
  int64_t local = i - c * s;
  if (c != r) {
    const int64_t first = R - r * s;  // rows of rank r's first chunk
    local += first < 0 ? 0 : (first > s ? s : first);
  }
  return RankRow{r, local};
}

// One destination rank: each of its rows fetched from where it sits at the
// source degree.
template <int kLanes, bool kStream>
__global__ __launch_bounds__(kThreads) void repartition_kernel(RepartitionParams p) {
  const int64_t t = row_index<kLanes>();
  if (t >= p.n_rows) return;
  const RankRow from = rank_row(row_position(p.dst_q_begin, p.dst_q_len, t) - p.P, p.C_src, p.s_src, p.R);
  copy_rows<kLanes, 1, kStream>({p.src[from.rank] + from.row * p.row_bytes}, {p.dst + t * p.row_bytes}, p.row_bytes,
                                threadIdx.x % kLanes);
}

// Every row of the suffix from its source rank to its destination rank, in
// kSets row sets at once.
template <int kLanes, int kSets, bool kStream>
__global__ __launch_bounds__(kThreads) void repartition_all_kernel(RepartitionAllParams p) {
  const int64_t i = row_index<kLanes>();
  if (i >= p.R) return;
  const RankRow from = rank_row(i, p.C_src, p.s_src, p.R);
  const RankRow to = rank_row(i, p.C_dst, p.s_dst, p.R);
  const unsigned char* src[kSets];
  unsigned char* dst[kSets];
#pragma unroll
  for (int s = 0; s < kSets; ++s) {
    src[s] = p.src[s][from.rank] + from.row * p.row_bytes;
    dst[s] = p.dst[s][to.rank] + to.row * p.row_bytes;
  }
  copy_rows<kLanes, kSets, kStream>(src, dst, p.row_bytes, threadIdx.x % kLanes);
}

// A block-table entry outside the cache gives zero rows.
template <int kLanes>
__global__ __launch_bounds__(kThreads) void kv_gather_kernel(GatherParams p) {
  const int64_t t = row_index<kLanes>();
  if (t >= p.n_rows) return;
  const int64_t pos = p.pos_begin + t;
  const int64_t blk = p.block_table[pos / kBlockTokens];
  const bool inside = blk >= 0 && blk < p.n_blocks;
  const int64_t src = (blk * kBlockTokens + pos % kBlockTokens) * p.row_bytes;
  copy_rows<kLanes, 2, true>({inside ? p.k_cache + src : nullptr, inside ? p.v_cache + src : nullptr},
                             {p.k_rows + t * p.row_bytes, p.v_rows + t * p.row_bytes}, p.row_bytes,
                             threadIdx.x % kLanes);
}

// Launches the kernel of the fewest lanes that hold a row's pieces one each.
template <class Params>
int launch_rows(void (*k16)(Params), void (*k32)(Params), void (*k64)(Params), const Params& p, int64_t rows,
                const char* who, void* stream) {
  if (rows == 0) return CP_OK;
  const int64_t pieces = p.row_bytes >> 4;
  const int lanes = pieces <= 16 ? 16 : pieces <= 32 ? 32 : 64;
  const int64_t per_block = kThreads / lanes;
  hipLaunchKernelGGL(lanes == 16 ? k16 : lanes == 32 ? k32 : k64, dim3((unsigned)((rows + per_block - 1) / per_block)),
                     dim3(kThreads), 0, (hipStream_t)stream, p);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(CP_ERR_HIP, std::string(who) + " launch: " + hipGetErrorString(e));
  return CP_OK;
}

}  // namespace

int launch_repartition_all(const RepartitionAllParams& p, void* stream) {
  const bool streamed = p.n_sets * p.R * p.row_bytes > kInfinityCacheBytes;
  auto launch = [&](auto k16, auto k32, auto k64) {
    return launch_rows<RepartitionAllParams>(k16, k32, k64, p, p.R, "cp_repartition_all", stream);
  };
  if (p.n_sets == 2)
    return streamed ? launch(repartition_all_kernel<16, 2, true>, repartition_all_kernel<32, 2, true>,
                             repartition_all_kernel<64, 2, true>)
                    : launch(repartition_all_kernel<16, 2, false>, repartition_all_kernel<32, 2, false>,
                             repartition_all_kernel<64, 2, false>);
  return streamed ? launch(repartition_all_kernel<16, 1, true>, repartition_all_kernel<32, 1, true>,
                           repartition_all_kernel<64, 1, true>)
                  : launch(repartition_all_kernel<16, 1, false>, repartition_all_kernel<32, 1, false>,
                           repartition_all_kernel<64, 1, false>);
}

int launch_gather(const GatherParams& p, void* stream) {
  return launch_rows(kv_gather_kernel<16>, kv_gather_kernel<32>, kv_gather_kernel<64>, p, p.n_rows, "cp_kv_gather",
                     stream);
}

int launch_writeback(const WritebackParams& p, void* stream) {
  if (2 * p.n_rows * p.row_bytes > kInfinityCacheBytes)
    return launch_rows(kv_writeback_kernel<16, true>, kv_writeback_kernel<32, true>, kv_writeback_kernel<64, true>, p,
                       p.n_rows, "cp_kv_writeback", stream);
  return launch_rows(kv_writeback_kernel<16, false>, kv_writeback_kernel<32, false>, kv_writeback_kernel<64, false>, p,
                     p.n_rows, "cp_kv_writeback", stream);
}

int launch_repartition(const RepartitionParams& p, void* stream) {
  if (p.n_rows * p.row_bytes > kInfinityCacheBytes)
    return launch_rows(repartition_kernel<16, true>, repartition_kernel<32, true>, repartition_kernel<64, true>, p,
                       p.n_rows, "cp_repartition", stream);
  return launch_rows(repartition_kernel<16, false>, repartition_kernel<32, false>, repartition_kernel<64, false>, p,
                     p.n_rows, "cp_repartition", stream);
}

}  // namespace cpattn
