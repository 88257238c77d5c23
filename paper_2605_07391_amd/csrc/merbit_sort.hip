// Scans and a stable radix-sort pass for the one-time plan work (column
// stripes, hot-column selection, the transpose of the adjoint).
//
// Scan: three launches over chunks of kScanChunk values -- each block reduces
// its chunk, one block scans the chunk totals, each block scans its chunk
// from its total's prefix.  Sum and max, inclusive or exclusive, int32.
//
// Radix pass: a stable counting sort of (key, value[, value]) records by the
// digit (key >> shift) & (2^bits - 1), bits <= 8.  A block owns kSortBlock
// consecutive records, each of its wavefronts a run of them.  A first launch
// counts the digits of every block; the counts, stored digit-major, are
// scanned; a second launch ranks the block's records by digit (the lanes that
// hold equal digits find each other with one ballot per digit bit, and the
// highest of them advances the wavefront's LDS counter), puts them in digit
// order in LDS and writes them from there, so that consecutive lanes write
// consecutive records of a digit's run.  Digit-major order of the counts keeps
// equal digits in block order, and ranks keep them in order inside a block, so
// the pass is stable.  LSD passes over successive digit fields sort by the
// whole key.
//
// What bounds it: the scattered runs (16 records of a digit per block at 8
// bits) against 12 or 20 bytes read and written per record.  Records written
// straight from the lanes (64 places per store) took 255 us per pass of 15.7M
// (column, position) pairs of R-MAT 20; reordered, with a third word per
// record, 111 us (145 us with an LDS array per word: three blocks per CU
// instead of five).  The count takes 19 us (49 us with a ballot per digit
// bit instead of LDS atomics).
#include <limits.h>

#include "merbit_internal.hpp"

namespace merbit {

// ------------------------------------------------------------------ scan --

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanChunk = kScanThreads * kScanItems;
constexpr int kPartThreads = 1024;

struct ScanSum {
  static __device__ __forceinline__ int32_t id() { return 0; }
  static __device__ __forceinline__ int32_t op(int32_t a, int32_t b) { return a + b; }
};
struct ScanMax {
  static __device__ __forceinline__ int32_t id() { return INT_MIN; }
  static __device__ __forceinline__ int32_t op(int32_t a, int32_t b) { return a > b ? a : b; }
};

// Inclusive scan over the block's threads (blockDim.x = THREADS, a multiple
// of 64); every thread gets its own inclusive value, *total the block's.
template <class Op, int THREADS>
__device__ __forceinline__ int32_t block_inclusive_scan(int32_t v, int32_t* s_wave,
                                                        int32_t* total) {
  const int lid = threadIdx.x & (kOmega - 1), wid = threadIdx.x / kOmega;
#pragma unroll
  for (int d = 1; d < kOmega; d <<= 1) {
    const int32_t t = __shfl_up(v, d, kOmega);
    if (lid >= d) v = Op::op(t, v);
  }
  if (lid == kOmega - 1) s_wave[wid] = v;
  __syncthreads();
  int32_t before = Op::id();
  int32_t all = Op::id();
  for (int w = 0; w < THREADS / kOmega; ++w) {
    if (w < wid) before = Op::op(before, s_wave[w]);
    all = Op::op(all, s_wave[w]);
  }
  __syncthreads();  // s_wave may be reused by the caller
  *total = all;
  return Op::op(before, v);
}

template <class Op>
__global__ __launch_bounds__(kScanThreads) void scan_reduce_kernel(const int32_t* __restrict__ in,
                                                                   int64_t n,
                                                                   int32_t* __restrict__ part) {
  __shared__ int32_t s_wave[kScanThreads / kOmega];
  const int64_t base = (int64_t)blockIdx.x * kScanChunk;
  int32_t acc = Op::id();
#pragma unroll
  for (int it = 0; it < kScanItems; ++it) {
    const int64_t i = base + it * kScanThreads + threadIdx.x;
    if (i < n) acc = Op::op(acc, in[i]);
  }
  int32_t total;
  (void)block_inclusive_scan<Op, kScanThreads>(acc, s_wave, &total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// part[0 .. nb) <- its exclusive scan (one block)
template <class Op>
__global__ __launch_bounds__(kPartThreads) void scan_parts_kernel(int32_t* __restrict__ part,
                                                                  int64_t nb) {
  __shared__ int32_t s_wave[kPartThreads / kOmega];
  __shared__ int32_t s_incl[kPartThreads];
  int32_t carry = Op::id();
  for (int64_t b0 = 0; b0 < nb; b0 += kPartThreads) {
    const int64_t b = b0 + threadIdx.x;
    const int32_t v = b < nb ? part[b] : Op::id();
    int32_t total;
    const int32_t incl = block_inclusive_scan<Op, kPartThreads>(v, s_wave, &total);
    s_incl[threadIdx.x] = incl;
    __syncthreads();
    const int32_t excl = threadIdx.x == 0 ? carry : Op::op(carry, s_incl[threadIdx.x - 1]);
    if (b < nb) part[b] = excl;
    carry = Op::op(carry, total);
    __syncthreads();
  }
}

// LDS index of chunk element i: one pad word per 16 keeps a thread's run of
// kScanItems consecutive elements on distinct banks across the wavefront
__device__ __forceinline__ int scan_lds(int i) { return i + (i >> 4); }

template <class Op, bool EXCLUSIVE>
__global__ __launch_bounds__(kScanThreads) void scan_apply_kernel(
    const int32_t* in, int32_t* out, int64_t n, const int32_t* __restrict__ part) {
  // in == out is allowed: the block reads its whole chunk before writing it
  __shared__ int32_t s[kScanChunk + kScanChunk / 16];
  __shared__ int32_t s_wave[kScanThreads / kOmega];
  const int64_t base = (int64_t)blockIdx.x * kScanChunk;
#pragma unroll
  for (int it = 0; it < kScanItems; ++it) {
    const int k = it * kScanThreads + threadIdx.x;
    s[scan_lds(k)] = base + k < n ? in[base + k] : Op::id();
  }
  __syncthreads();
  const int first = threadIdx.x * kScanItems;
  int32_t run = Op::id();
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) run = Op::op(run, s[scan_lds(first + k)]);
  int32_t total;
  const int32_t incl = block_inclusive_scan<Op, kScanThreads>(run, s_wave, &total);
  // everything before this thread's run: the chunk's prefix and the previous
  // thread's inclusive value (max has no inverse, so no subtraction)
  __shared__ int32_t s_prev[kScanThreads];
  s_prev[threadIdx.x] = incl;
  __syncthreads();
  int32_t acc =
      threadIdx.x == 0 ? part[blockIdx.x] : Op::op(part[blockIdx.x], s_prev[threadIdx.x - 1]);
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int li = scan_lds(first + k);
    const int32_t v = s[li];
    if (EXCLUSIVE) {
      s[li] = acc;
      acc = Op::op(acc, v);
    } else {
      acc = Op::op(acc, v);
      s[li] = acc;
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kScanItems; ++it) {
    const int k = it * kScanThreads + threadIdx.x;
    if (base + k < n) out[base + k] = s[scan_lds(k)];
  }
}

int64_t scan_blocks(int64_t n) { return (n + kScanChunk - 1) / kScanChunk; }

size_t scan_temp_bytes(int64_t n) {
  return sizeof(int32_t) * (size_t)(scan_blocks(n) > 0 ? scan_blocks(n) : 1);
}

template <class Op, bool EXCLUSIVE>
static hipError_t scan_t(const int32_t* in, int32_t* out, int64_t n, int32_t* part,
                         hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t nb = scan_blocks(n);
  hipLaunchKernelGGL((scan_reduce_kernel<Op>), dim3((unsigned)nb), dim3(kScanThreads), 0, st, in,
                     n, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((scan_parts_kernel<Op>), dim3(1), dim3(kPartThreads), 0, st, part, nb);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL((scan_apply_kernel<Op, EXCLUSIVE>), dim3((unsigned)nb), dim3(kScanThreads),
                     0, st, in, out, n, part);
  return hipGetLastError();
}

hipError_t launch_scan_i32(const int32_t* in, int32_t* out, int64_t n, ScanKind kind,
                           void* temp, hipStream_t st) {
  int32_t* part = static_cast<int32_t*>(temp);
  switch (kind) {
    case kScanExclusiveSum: return scan_t<ScanSum, true>(in, out, n, part, st);
    case kScanInclusiveSum: return scan_t<ScanSum, false>(in, out, n, part, st);
    case kScanInclusiveMax: return scan_t<ScanMax, false>(in, out, n, part, st);
  }
  return hipErrorInvalidValue;
}

// ------------------------------------------------------------ radix pass --

constexpr int kSortWaves = 4;
constexpr int kSortThreads = kSortWaves * kOmega;
constexpr int kSortItems = 16;  // records per thread (8: level; 32: 15 % slower)
constexpr int kSortRun = kOmega * kSortItems;
constexpr int kSortBlock = kSortWaves * kSortRun;
constexpr int kSortMaxDigits = 256;
static_assert(kSortThreads == kSortMaxDigits, "one thread per digit");

// Lanes of the wavefront whose `valid` digit equals this lane's.
__device__ __forceinline__ unsigned long long digit_peers(uint32_t d, bool valid, int bits) {
  unsigned long long m = __ballot(valid);
  for (int b = 0; b < bits; ++b) {
    const bool on = (d >> b) & 1u;
    const unsigned long long bal = __ballot(valid && on);
    m &= on ? bal : ~bal;
  }
  return m;
}

// counts[d * nblk + b] = records of digit d in block b
__global__ __launch_bounds__(kSortThreads) void radix_count_kernel(
    const uint32_t* __restrict__ key, int64_t n, int shift, int bits, int64_t nblk,
    int32_t* __restrict__ counts) {
  // one set of counters per wavefront: equal digits of a wavefront meet anyway
  __shared__ int32_t s_cnt[kSortWaves][kSortMaxDigits];
  const int tid = threadIdx.x, wid = tid / kOmega;
  const uint32_t dmask = (1u << bits) - 1u;
  for (int w = 0; w < kSortWaves; ++w) s_cnt[w][tid] = 0;
  const int64_t base = (int64_t)blockIdx.x * kSortBlock;
  uint32_t k[kSortItems];
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    const int64_t i = base + it * kSortThreads + tid;
    k[it] = i < n ? key[i] : 0u;
  }
  __syncthreads();
  if (bits <= 4) {
    // few digits: a wavefront's lanes would meet on a few counters (3 bits,
    // R-MAT 22: 174 us with atomics)
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
      const bool valid = base + it * kSortThreads + tid < n;
      const uint32_t d = (k[it] >> shift) & dmask;
      const unsigned long long peers = digit_peers(d, valid, bits);
      if (valid && 63 - __builtin_clzll(peers) == (tid & (kOmega - 1)))
        s_cnt[wid][d] += __popcll(peers);
      wave_lds_sync();
    }
  } else {
#pragma unroll
    for (int it = 0; it < kSortItems; ++it)
      if (base + it * kSortThreads + tid < n) atomicAdd(&s_cnt[wid][(k[it] >> shift) & dmask], 1);
  }
  __syncthreads();
  if (tid <= (int)dmask) {
    int32_t c = 0;
    for (int w = 0; w < kSortWaves; ++w) c += s_cnt[w][tid];
    counts[(int64_t)tid * nblk + blockIdx.x] = c;
  }
}

template <bool TWO>
__global__ __launch_bounds__(kSortThreads) void radix_scatter_kernel(
    const uint32_t* __restrict__ key_in, const int32_t* __restrict__ val_in,
    const int32_t* __restrict__ val2_in, uint32_t* __restrict__ key_out,
    int32_t* __restrict__ val_out, int32_t* __restrict__ val2_out, int64_t n, int shift, int bits,
    int64_t nblk, const int32_t* __restrict__ offsets) {
  __shared__ uint32_t s_rec[kSortBlock];  // the keys, then each value, in digit order
  __shared__ int32_t s_cnt[kSortWaves][kSortMaxDigits];
  __shared__ int32_t s_goff[kSortMaxDigits];
  __shared__ int32_t s_wave[kSortWaves];
  const int tid = threadIdx.x, lid = tid & (kOmega - 1), wid = tid / kOmega;
  const uint32_t dmask = (1u << bits) - 1u;
  for (int w = 0; w < kSortWaves; ++w) s_cnt[w][tid] = 0;
  const int64_t base = (int64_t)blockIdx.x * kSortBlock;
  const int n_blk = (int)(n - base < kSortBlock ? n - base : kSortBlock);
  const int first = wid * kSortRun + lid;  // this thread's records: first + 64 it
  uint32_t k[kSortItems];
  int32_t v[kSortItems], v2[kSortItems];  // v2 only with TWO
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    const int q = first + it * kOmega;
    k[it] = q < n_blk ? key_in[base + q] : 0u;
  }
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    const int q = first + it * kOmega;
    v[it] = val_in == nullptr ? (int32_t)(base + q) : (q < n_blk ? val_in[base + q] : 0);
    if constexpr (TWO) v2[it] = q < n_blk ? val2_in[base + q] : 0;
  }
  __syncthreads();
  // rank among the wavefront's records of the same digit
  const unsigned long long below = (1ull << lid) - 1ull;
  int32_t* cnt = s_cnt[wid];
  int rank[kSortItems];
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    const bool valid = first + it * kOmega < n_blk;
    const uint32_t d = (k[it] >> shift) & dmask;
    const unsigned long long peers = digit_peers(d, valid, bits);
    const int32_t before = cnt[d];
    rank[it] = before + __popcll(peers & below);
    wave_lds_sync();  // every lane has read its digit's count
    if (valid && 63 - __builtin_clzll(peers) == lid) cnt[d] = before + __popcll(peers);
    wave_lds_sync();
  }
  __syncthreads();
  // thread d: where digit d begins in the block, and each wavefront's part
  int32_t c = 0;
#pragma unroll
  for (int w = 0; w < kSortWaves; ++w) {
    const int32_t own = s_cnt[w][tid];
    s_cnt[w][tid] = c;
    c += own;
  }
  int32_t total;
  const int32_t start = block_inclusive_scan<ScanSum, kSortThreads>(c, s_wave, &total) - c;
#pragma unroll
  for (int w = 0; w < kSortWaves; ++w) s_cnt[w][tid] += start;
  if (tid <= (int)dmask) s_goff[tid] = offsets[(int64_t)tid * nblk + blockIdx.x] - start;
  __syncthreads();
  // rank becomes the record's place in the block's digit order
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    rank[it] += cnt[(k[it] >> shift) & dmask];
    if (first + it * kOmega < n_blk) s_rec[rank[it]] = k[it];
  }
  __syncthreads();
  int32_t to[kSortItems];  // where the block's record tid + 256 it goes
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    const int q = tid + it * kSortThreads;
    if (q < n_blk) {
      const uint32_t key = s_rec[q];
      to[it] = s_goff[(key >> shift) & dmask] + q;
      key_out[to[it]] = key;
    }
  }
  auto put = [&](const int32_t (&x)[kSortItems], int32_t* __restrict__ out) {
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kSortItems; ++it)
      if (first + it * kOmega < n_blk) s_rec[rank[it]] = (uint32_t)x[it];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kSortItems; ++it) {
      const int q = tid + it * kSortThreads;
      if (q < n_blk) out[to[it]] = (int32_t)s_rec[q];
    }
  };
  put(v, val_out);
  if constexpr (TWO) put(v2, val2_out);
}

static int64_t sort_blocks(int64_t n) { return (n + kSortBlock - 1) / kSortBlock; }

size_t radix_temp_bytes(int64_t n, int bits) {
  const int64_t counts = sort_blocks(n) * ((int64_t)1 << bits);
  return sizeof(int32_t) * (size_t)(counts > 0 ? counts : 1) + scan_temp_bytes(counts) + 256;
}

hipError_t launch_radix_pass(const uint32_t* key_in, const int32_t* val_in, uint32_t* key_out,
                             int32_t* val_out, int64_t n, int shift, int bits, void* temp,
                             hipStream_t st, const int32_t* val2_in, int32_t* val2_out) {
  if (n <= 0) return hipSuccess;
  if (bits < 1 || bits > 8) return hipErrorInvalidValue;
  const int64_t nblk = sort_blocks(n);
  const int64_t nc = nblk * ((int64_t)1 << bits);
  int32_t* counts = static_cast<int32_t*>(temp);
  int32_t* part = reinterpret_cast<int32_t*>(
      static_cast<unsigned char*>(temp) + ((sizeof(int32_t) * (size_t)nc + 255) & ~(size_t)255));
  const dim3 grid((unsigned)nblk), block(kSortThreads);
  hipLaunchKernelGGL(radix_count_kernel, grid, block, 0, st, key_in, n, shift, bits, nblk, counts);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_scan_i32(counts, counts, nc, kScanExclusiveSum, part, st);
  if (e != hipSuccess) return e;
  if (val2_in != nullptr)
    hipLaunchKernelGGL((radix_scatter_kernel<true>), grid, block, 0, st, key_in, val_in, val2_in,
                       key_out, val_out, val2_out, n, shift, bits, nblk, counts);
  else
    hipLaunchKernelGGL((radix_scatter_kernel<false>), grid, block, 0, st, key_in, val_in, val2_in,
                       key_out, val_out, val2_out, n, shift, bits, nblk, counts);
  return hipGetLastError();
}

}  // namespace merbit
