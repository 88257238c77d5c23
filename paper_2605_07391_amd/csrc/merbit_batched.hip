// Batched forms on the same plan: Y = A X for up to 64 right-hand sides at
// once, the per-column PageRank update for personalised PageRank, and the
// per-graph PageRank update for many graphs stored on the diagonal of one
// matrix.
//
// SpMM (one wavefront per tile; the driver runs one launch per slab of 32
// columns).  The tile's merge-path segment (Sec. 4.1) fixes its nonzeros
// [x_ws, x_we) and rows [y_ws, y_we]; every nonzero is a row operation
// Y[row, :] += v * X[col, :].  A lane carries W columns (one 16-byte access
// where the operands' alignment allows it); the wavefront is cut into groups
// of KP lanes, KP the power of two that holds the slab's columns, and each
// group takes an equal run of the tile's nonzeros:
//   1. the tile's values, X row offsets and rows (decoded from the lane
//      descriptors, Sec. 4.1.1) go to LDS;
//   2. each group walks its run, kSpmmUnroll X rows in flight before the first
//      is used; a row that begins and ends inside the run is complete, the
//      run's first and last rows are not;
//   3. a head-flagged segmented scan over the groups completes those;
//   4. the empty rows inside the tile are written as 0.
// Rows strictly inside the tile are stored; the tile's first and last rows
// (shared with neighbouring tiles) are added atomically to Y, which is zero
// there before the launch.
//
// What bounds it: on large graphs the X row reads that miss L2 (R-MAT 20, 32
// columns, FP32: 2 GB of them in 238 us); otherwise the instructions per
// nonzero, which the groups divide by 64 / KP.  A wavefront that walks one
// nonzero at a time, its idle lanes repeating the last column, takes as long
// for 1 column as for 32.  R-MAT 18, 2 / 8 / 16 / 32 columns, one nonzero at a
// time, then groups of one column per lane, then several columns per lane:
// FP32 102 / 103 / 103 / 103, 44 / 51 / 64 / 96, 42 / 46 / 48 / 55 us; FP64
// 153 / 154 / 154 / 160, 45 / 51 / 64 / 107, 44 / 50 / 51 / 103 us.  sigma is an argument, not a template parameter: only the staging
// loops depend on it.
#include "merbit_internal.hpp"

namespace merbit {

constexpr int kSpmmWaves = 4;
// X rows in flight per group before the first is used: 16 loads of one column
// per lane (R-MAT 18 FP32, 32 columns: 129 / 105 / 95 us at 4 / 8 / 16), 8 of
// several (61 / 55 / 53 us; FP64 100 / 103 / 105 us, 8 columns on Chung-Lu
// 700,001 88 / 86 / 99 us)
constexpr int kSpmmUnroll = 16;
constexpr int kSpmmUnrollWide = 8;
// word 3 of a raw (unformatted, stride 0) buffer resource on gfx950
constexpr int kSpmmBufferWord3 = 0x00020000;

// W consecutive columns of a row
template <typename V, int W>
struct Cols {
  typedef V type __attribute__((ext_vector_type(W)));
};

// Per-lane state of a fused personalised-PageRank step (SpmmArgs::Xn).
template <typename V, int W>
struct PprRow {
  V* Xn;
  int64_t ld;
  V a;                 // alpha
  V tele[W];           // alpha delta_j + 1 - alpha, added at the column's source row
  int sj[W];           // the column's source row (-1: lane past the slab)
  int w0;              // dmask word of the tile's first row
  const uint32_t* dm;  // the tile's dmask words (LDS)
  double dsum[W];      // dangling mass of the rows this lane finished
};

// Columns j .. j + W - 1 of row y_ws + rel are complete.  The tile's first and
// last rows are shared with neighbouring tiles and are added to Y; the others
// are stored, or with FUSE finished as the next iterate.
template <typename V, int W, bool FUSE>
__device__ __forceinline__ void spmm_row(const SpmmArgs& a, int j, int y_ws, int rel,
                                         int last_rel, typename Cols<V, W>::type acc,
                                         PprRow<V, W>& f) {
  typedef typename Cols<V, W>::type VW;
  const int row = y_ws + rel;
  V* y = static_cast<V*>(a.Y) + (int64_t)row * a.ldy + j;
  if (rel == 0 || rel == last_rel) {
    if (row < a.n_rows)
#pragma unroll
      for (int c = 0; c < W; ++c) global_add(y + c, acc[c]);
  } else if constexpr (FUSE) {
    VW xn;
    const bool dangling = (f.dm[(row >> 5) - f.w0] >> (row & 31)) & 1u;
#pragma unroll
    for (int c = 0; c < W; ++c) {
      V v = f.a * acc[c];
      if (row == f.sj[c]) v += f.tele[c];
      xn[c] = v;
      if (dangling) f.dsum[c] += (double)v;
    }
    __builtin_nontemporal_store(xn, reinterpret_cast<VW*>(f.Xn + (int64_t)row * f.ld + j));
  } else {
    // written once, not read here again
    __builtin_nontemporal_store(acc, reinterpret_cast<VW*>(y));
  }
}

// LDS bytes of one wavefront: the tile's values, X row offsets, rows and the
// marks of its non-empty rows, and (fused step) its dmask words.
template <typename V>
static __host__ __device__ constexpr int spmm_wave_lds(int sigma) {
  return kOmega * sigma * ((int)sizeof(V) + 4 + 2 + 1) + kOmega * 4;
}

// KP lanes per group, W columns per lane: KP W >= a.k, a.k a multiple of W.
template <typename V, int KP, int W, bool FUSE>
__global__ __launch_bounds__(kSpmmWaves * 64) void spmm_kernel(SpmmArgs a, int sigma) {
  typedef typename Cols<V, W>::type VW;
  constexpr int G = kOmega / KP;  // groups of KP lanes
  constexpr int U = W == 1 ? kSpmmUnroll : kSpmmUnrollWide;
  extern __shared__ __align__(16) unsigned char s_dyn[];
  const int lid = threadIdx.x & (kOmega - 1);
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kOmega);
  const int g = lid / KP, j = lid % KP * W;
  const int t = blockIdx.x * kSpmmWaves + wid;
  const bool on = j < a.k;
  PprRow<V, W> f{};
  if constexpr (FUSE) {
    f.Xn = static_cast<V*>(a.Xn);
    f.ld = a.ldx;
    f.a = (V)a.alpha;
#pragma unroll
    for (int c = 0; c < W; ++c) {
      f.sj[c] = on ? a.src[j + c] : -1;
      f.tele[c] = on ? (V)(a.alpha * a.sums_in[2 * (j + c)] + 1.0 - a.alpha) : V(0);
      f.dsum[c] = 0.0;
    }
  }
  if (t < a.tile_num) {
    const int T = kOmega * sigma;
    unsigned char* lds = s_dyn + wid * spmm_wave_lds<V>(sigma);
    V* s_val = reinterpret_cast<V*>(lds);
    uint32_t* s_off = reinterpret_cast<uint32_t*>(s_val + T);
    uint32_t* s_dm = s_off + T;
    uint16_t* s_row = reinterpret_cast<uint16_t*>(s_dm + kOmega);
    unsigned char* s_has = reinterpret_cast<unsigned char*>(s_row + T);

    const int x_ws = a.tile_x[t];
    const int x_se = a.tile_x[t + 1] - x_ws;
    const uint32_t tyw = a.tile_y[t];
    const int y_ws = (int)(tyw & kRowMask);
    const int last_rel = (int)(a.tile_y[t + 1] & kRowMask) - y_ws;
    const V* __restrict__ X = static_cast<const V*>(a.X);
    const uint32_t row_bytes = (uint32_t)(a.ldx * (int64_t)sizeof(V));
    const bool buf = a.x_rows * a.ldx * (int64_t)sizeof(V) < ((int64_t)1 << 31);

    // 1. the tile into LDS.  The matrix stream is read once: non-temporal, so
    // it does not push the reused X rows out of L2.
    for (int q = lid; q < x_se; q += kOmega) {
      const int c = __builtin_nontemporal_load(a.col + x_ws + q);
      s_val[q] = __builtin_nontemporal_load(static_cast<const V*>(a.val) + x_ws + q);
      s_off[q] = buf ? (uint32_t)c * row_bytes : (uint32_t)c;
    }
    for (int q = lid; q < T / 4; q += kOmega) reinterpret_cast<uint32_t*>(s_has)[q] = 0u;
    if constexpr (FUSE) {
      // the tile's rows y_ws .. y_ws + last_rel span at most 2 sigma + 2 words
      f.w0 = y_ws >> 5;
      f.dm = s_dm;
      s_dm[lid] = f.w0 + lid < a.dmask_words ? a.dmask[f.w0 + lid] : 0u;
    }
    tile_nz_rows(a.lane_desc, a.lane_num, a.path_len, sigma, t, tyw, x_se, lid, s_row);
    wave_lds_sync();
    for (int q = lid; q < x_se; q += kOmega) s_has[s_row[q]] = 1;
    wave_lds_sync();

    // 2. group g walks nonzeros [g L, (g + 1) L), its lanes the columns.  cur
    // is the row of the nonzero before them: the first row change ends a row
    // that groups before this one may have begun, so its sum waits in `first`
    // for their carry; every later row is complete.
    const int L = ((x_se + G - 1) / G + U - 1) / U * U;
    const int q0 = g * L;
    const int cnt = min(max(x_se - q0, 0), L);
    int cur0 = 0, cur = 0;
    bool has = false;
    VW acc = VW(0), first = VW(0);
    if (cnt > 0) cur0 = cur = s_row[q0 > 0 ? q0 - 1 : 0];
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        (void*)X, (short)0,
        buf ? (int)(((a.x_rows - 1) * a.ldx + a.k) * (int64_t)sizeof(V)) : 0, kSpmmBufferWord3);
    const int jx = min(j, a.k - W);  // lanes past k read the row's last columns again
    auto walk = [&](auto load) {
      for (int i = 0; i < cnt; i += U) {
        uint32_t off[U];
        V v[U];
        VW x[U];
        uint16_t r[U];
        const int q = q0 + i;  // a multiple of U: aligned vector reads
#pragma unroll
        for (int u = 0; u < U; ++u) {
          off[u] = s_off[q + u];
          v[u] = s_val[q + u];
          r[u] = s_row[q + u];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = load(i + u < cnt ? off[u] : off[0]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (i + u < cnt) {
            if ((int)r[u] != cur) {
              if (!has) first = acc;
              else if (on) spmm_row<V, W, FUSE>(a, j, y_ws, cur, last_rel, acc, f);
              has = true;
              cur = r[u];
              acc = VW(0);
            }
#pragma unroll
            for (int c = 0; c < W; ++c) acc[c] += v[u] * x[u][c];
          }
        }
      }
    };
    if (buf) {
      walk([&](uint32_t off) -> VW {
        const int at = (int)off + jx * (int)sizeof(V);
        if constexpr (sizeof(VW) == 4)
          return __builtin_bit_cast(VW, __builtin_amdgcn_raw_buffer_load_b32(rx, at, 0, 0));
        else if constexpr (sizeof(VW) == 8)
          return __builtin_bit_cast(VW, __builtin_amdgcn_raw_buffer_load_b64(rx, at, 0, 0));
        else
          return __builtin_bit_cast(VW, __builtin_amdgcn_raw_buffer_load_b128(rx, at, 0, 0));
      });
    } else {
      walk([&](uint32_t c) -> VW {
        return *reinterpret_cast<const VW*>(X + (int64_t)c * a.ldx + jx);
      });
    }
    // 3. the groups' carries: a segmented scan over the groups of a column
    VW sum = acc;
    int head = has;
#pragma unroll
    for (int d = KP; d < kOmega; d <<= 1) {
      VW ts;
#pragma unroll
      for (int c = 0; c < W; ++c) ts[c] = __shfl_up(sum[c], d, kOmega);
      const int th = __shfl_up(head, d, kOmega);
      if (lid >= d) {
        if (!head) sum += ts;
        head |= th;
      }
    }
    VW carry;
#pragma unroll
    for (int c = 0; c < W; ++c) carry[c] = __shfl_up(sum[c], KP, kOmega);
    if (g == 0) carry = VW(0);
    if (has && on) spmm_row<V, W, FUSE>(a, j, y_ws, cur0, last_rel, first + carry, f);
    if (x_se > 0 && g == G - 1 && on)
      spmm_row<V, W, FUSE>(a, j, y_ws, s_row[x_se - 1], last_rel, sum, f);
    // 4. the empty rows strictly inside the tile
    for (int e = 1 + g; e < last_rel; e += G)
      if (!s_has[e] && on) spmm_row<V, W, FUSE>(a, j, y_ws, e, last_rel, VW(0), f);
    if (a.Z != nullptr && g == 0 && on)
      *reinterpret_cast<VW*>(static_cast<V*>(a.Z) + (int64_t)y_ws * a.ldz + j) = VW(0);
  }
  if constexpr (FUSE) {
    // the block's dangling mass per column: its wavefronts and groups in order
    __shared__ double s_d[kSpmmWaves * kOmega * W];
#pragma unroll
    for (int c = 0; c < W; ++c) s_d[threadIdx.x * W + c] = f.dsum[c];
    __syncthreads();
    if (threadIdx.x < a.k) {
      double d = 0.0;
      for (int w = 0; w < kSpmmWaves * G; ++w) d += s_d[w * KP * W + threadIdx.x];
      double* o = a.part + ((int64_t)blockIdx.x * kOmega + a.col0 + threadIdx.x) * 2;
      o[0] = d;
      o[1] = 0.0;
    }
  }
}

int spmm_blocks(int64_t tile_num) { return (int)((tile_num + kSpmmWaves - 1) / kSpmmWaves); }

template <typename V, int KP, int W>
static hipError_t spmm_launch_t(const SpmmArgs& a, int sigma, hipStream_t st) {
  const unsigned grid = (unsigned)spmm_blocks(a.tile_num);
  const size_t lds = (size_t)kSpmmWaves * spmm_wave_lds<V>(sigma);
  if (a.Xn != nullptr)
    hipLaunchKernelGGL((spmm_kernel<V, KP, W, true>), dim3(grid), dim3(kSpmmWaves * 64), lds, st,
                       a, sigma);
  else
    hipLaunchKernelGGL((spmm_kernel<V, KP, W, false>), dim3(grid), dim3(kSpmmWaves * 64), lds, st,
                       a, sigma);
  return hipGetLastError();
}

// Columns per lane: as many as one 16-byte access holds, if every row of every
// operand allows it, so that a group needs fewer lanes.
template <typename V>
static bool spmm_wide(const SpmmArgs& a, int w) {
  const uintptr_t mask = (uintptr_t)w * sizeof(V) - 1;
  auto at = [&](const void* p, int64_t ld) {
    return p == nullptr || ((reinterpret_cast<uintptr_t>(p) & mask) == 0 && ld % w == 0);
  };
  return a.k % w == 0 && at(a.X, a.ldx) && at(a.Y, a.ldy) && at(a.Z, a.ldz) && at(a.Xn, a.ldx);
}

template <typename V, int W>
static hipError_t spmm_pick(const SpmmArgs& a, int sigma, hipStream_t st) {
  const int lanes = a.k / W;
  if (lanes <= 1) return spmm_launch_t<V, 1, W>(a, sigma, st);
  if (lanes <= 2) return spmm_launch_t<V, 2, W>(a, sigma, st);
  if (lanes <= 4) return spmm_launch_t<V, 4, W>(a, sigma, st);
  if (lanes <= 8) return spmm_launch_t<V, 8, W>(a, sigma, st);
  if constexpr (W <= 2)
    if (lanes <= 16) return spmm_launch_t<V, 16, W>(a, sigma, st);
  if constexpr (W == 1) return spmm_launch_t<V, 32, W>(a, sigma, st);
  return hipErrorInvalidValue;
}

hipError_t launch_spmm(int dtype, int sigma, const SpmmArgs& a, hipStream_t st) {
  if (a.tile_num == 0) return hipSuccess;
  if (sigma < 1 || sigma > kMaxSigma || a.k < 1 || a.k > kSlab) return hipErrorInvalidValue;
  if (dtype == 0) {
    if (spmm_wide<float>(a, 4)) return spmm_pick<float, 4>(a, sigma, st);
    if (spmm_wide<float>(a, 2)) return spmm_pick<float, 2>(a, sigma, st);
    return spmm_pick<float, 1>(a, sigma, st);
  }
  if (spmm_wide<double>(a, 2)) return spmm_pick<double, 2>(a, sigma, st);
  return spmm_pick<double, 1>(a, sigma, st);
}

// Zero Y[tile_y[t], col0 .. col0 + k) for every tile t (the rows the SpMM adds onto).
template <typename V>
__global__ void spmm_zero_kernel(const uint32_t* __restrict__ tile_y, int32_t tile_num, V* Y,
                                 int64_t ld, int k) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t t = e / 64, j = e % 64;
  if (t < tile_num && j < k) Y[(int64_t)(tile_y[t] & kRowMask) * ld + j] = V(0);
}

hipError_t launch_spmm_zero(int dtype, const uint32_t* tile_y, int32_t tile_num, void* Y,
                            int64_t ld, int k, hipStream_t st) {
  if (tile_num == 0) return hipSuccess;
  const unsigned grid = (unsigned)(((int64_t)tile_num * 64 + 255) / 256);
  if (dtype == 0)
    hipLaunchKernelGGL(spmm_zero_kernel<float>, dim3(grid), dim3(256), 0, st, tile_y, tile_num,
                       static_cast<float*>(Y), ld, k);
  else
    hipLaunchKernelGGL(spmm_zero_kernel<double>, dim3(grid), dim3(256), 0, st, tile_y, tile_num,
                       static_cast<double*>(Y), ld, k);
  return hipGetLastError();
}

// ---------------------------------------------- personalised PageRank step --
//
// Column j of X is the rank vector of source src[j]:
//   X'[r, j] = alpha Y[r, j] + (r == src[j]) (alpha delta_j + 1 - alpha),
// with delta_j the dangling mass of column j and Y = A X.  The SpMM finishes
// every row strictly inside a tile as X' itself (SpmmArgs::Xn) and adds its
// dangling mass to a per-block, per-column part; ppr_fixup_kernel finishes
// the tiles' first rows from Y (where neighbouring tiles added into them)
// and clears those slots of Y for the next step; on the last step of a
// chunk ppr_resid_kernel adds the l1 change.  A last kernel (one block per
// column) sums the parts in a fixed order for the next step and the host.
// Thread t of the part kernels always handles column t % K, K the power of two
// from k on, so each wavefront reads and writes 64 / K whole rows (coalesced;
// with column t % 64 the dangling, l1 and fixup kernels took 17.8, 13.4 and
// 8.2 us on R-MAT 18 FP32, k = 16, with 64 / K rows a wavefront 6.7, 7.1 and
// 4.9).
//
// The iterates (and A X) are held as slabs of kSlab columns one after
// another: slab s is the row-major n x W_s block of columns 32 s .. 32 s +
// W_s - 1 (W_s = min(32, k - 32 s)), so every SpMM launch reads and writes a
// compact array (for k <= 32 this is the row-major n x k layout).  Compact
// slabs took the 64-column SpMM of R-MAT 22 from 2.51 to 2.34 ms (FP32)
// against the two halves of a row-major n x 64 array.

// offset of element (r, j) of an n x k iterate in the slab layout
__device__ __forceinline__ int64_t ppr_at(int64_t r, int j, int64_t n, int k) {
  const int c0 = j & ~(kSlab - 1);
  const int w = min(kSlab, k - c0);
  return (int64_t)c0 * n + r * w + (j - c0);
}

constexpr int kPprThreads = 256;
constexpr int kPprWaves = kPprThreads / 64;
constexpr int kPprRows = 4;

// log2 of the columns K that a part kernel's lanes span
__device__ __forceinline__ int ppr_log_cols(int k) { return k > 1 ? 32 - __builtin_clz(k - 1) : 0; }

// per-thread (a, b) pairs of the block (thread t: column t % 2^ks) summed over
// each wavefront's rows in a fixed tree, then over the wavefronts in order, and
// written as part_out row blockIdx.x
__device__ __forceinline__ void ppr_block_part(double a, double b, double* __restrict__ part_out,
                                               int ks = 6) {
  __shared__ double s_a[kPprThreads], s_b[kPprThreads];
  for (int off = 32; off >= (1 << ks); off >>= 1) {
    a += __shfl_xor(a, off, kOmega);
    b += __shfl_xor(b, off, kOmega);
  }
  s_a[threadIdx.x] = a;
  s_b[threadIdx.x] = b;
  __syncthreads();
  if (threadIdx.x < 64) {
    double x = 0.0, y = 0.0;
    for (int q = 0; q < kPprWaves; ++q) {
      x += s_a[q * 64 + threadIdx.x];
      y += s_b[q * 64 + threadIdx.x];
    }
    part_out[((int64_t)blockIdx.x * 64 + threadIdx.x) * 2] = x;
    part_out[((int64_t)blockIdx.x * 64 + threadIdx.x) * 2 + 1] = y;
  }
}

int ppr_fixup_grid(int64_t tile_num) {
  int64_t g = (tile_num + kPprWaves * 8 - 1) / (kPprWaves * 8);
  if (g > 4096) g = 4096;
  if (g < 1) g = 1;
  return (int)g;
}

template <typename V>
__global__ __launch_bounds__(kPprThreads) void ppr_fixup_kernel(
    const uint32_t* __restrict__ tile_y, int32_t tile_num, V* __restrict__ Y,
    V* __restrict__ Xn, int64_t n, int k, double alpha, const int32_t* __restrict__ src,
    const double* __restrict__ sums_in, const uint32_t* __restrict__ dmask,
    double* __restrict__ part_out) {
  const int ks = ppr_log_cols(k);
  const int j = threadIdx.x & ((1 << ks) - 1);
  const int w = threadIdx.x >> ks;
  const bool on = j < k;
  const int sj = on ? src[j] : -1;
  const V a = (V)alpha;
  const V tele = on ? (V)(alpha * sums_in[2 * j] + 1.0 - alpha) : V(0);
  double dsum = 0.0;
  const int64_t step = (int64_t)gridDim.x * (kPprThreads >> ks);
  for (int64_t t = (int64_t)blockIdx.x * (kPprThreads >> ks) + w; t < tile_num; t += step) {
    const int64_t r = tile_y[t] & kRowMask;
    // each first row once (a long row is the first row of several tiles)
    if (r >= n || (t > 0 && (int64_t)(tile_y[t - 1] & kRowMask) == r)) continue;
    if (on) {
      const int64_t e = ppr_at(r, j, n, k);
      V xn = a * Y[e];
      Y[e] = V(0);
      if (r == sj) xn += tele;
      Xn[e] = xn;
      if ((dmask[r >> 5] >> (r & 31)) & 1u) dsum += (double)xn;
    }
  }
  ppr_block_part(dsum, 0.0, part_out, ks);
}

template <typename V>
__global__ __launch_bounds__(kPprThreads) void ppr_resid_kernel(const V* __restrict__ Xn,
                                                                const V* __restrict__ Xo,
                                                                int64_t n, int k,
                                                                double* __restrict__ part_out) {
  const int ks = ppr_log_cols(k);
  const int j = threadIdx.x & ((1 << ks) - 1);
  const int rb = kPprThreads >> ks;  // rows per pass of the block
  double rsum = 0.0;
  const int64_t step = (int64_t)gridDim.x * rb * kPprRows;
  for (int64_t r0 = (int64_t)blockIdx.x * rb * kPprRows + (threadIdx.x >> ks); j < k && r0 < n;
       r0 += step) {
    V xn[kPprRows], xo[kPprRows];
#pragma unroll
    for (int u = 0; u < kPprRows; ++u) {
      const int64_t e = ppr_at(min(r0 + u * rb, n - 1), j, n, k);
      xn[u] = Xn[e];
      xo[u] = Xo[e];
    }
#pragma unroll
    for (int u = 0; u < kPprRows; ++u)
      if (r0 + u * rb < n) rsum += fabs((double)xn[u] - (double)xo[u]);
  }
  ppr_block_part(0.0, rsum, part_out, ks);
}

// dangling mass of X (per column) -> the same per-block part layout
template <typename V>
__global__ __launch_bounds__(kPprThreads) void ppr_dangling_kernel(
    const V* __restrict__ X, const uint32_t* __restrict__ dmask, int64_t n, int k,
    double* __restrict__ part_out) {
  const int ks = ppr_log_cols(k);
  const int j = threadIdx.x & ((1 << ks) - 1);
  const int rb = kPprThreads >> ks;  // rows per pass of the block
  double dsum = 0.0;
  const int64_t step = (int64_t)gridDim.x * rb * kPprRows;
  for (int64_t r0 = (int64_t)blockIdx.x * rb * kPprRows + (threadIdx.x >> ks); j < k && r0 < n;
       r0 += step) {
    V v[kPprRows];
    uint32_t mw[kPprRows];
#pragma unroll
    for (int u = 0; u < kPprRows; ++u) {
      const int64_t r = min(r0 + u * rb, n - 1);
      v[u] = X[ppr_at(r, j, n, k)];
      mw[u] = dmask[r >> 5];
    }
#pragma unroll
    for (int u = 0; u < kPprRows; ++u) {
      const int64_t r = r0 + u * rb;
      if (r < n && ((mw[u] >> (r & 31)) & 1u)) dsum += (double)v[u];
    }
  }
  ppr_block_part(dsum, 0.0, part_out, ks);
}

// the slab layout back into the caller's row-major n x k (ld k), one
// wavefront per row
template <typename V>
__global__ __launch_bounds__(kPprThreads) void ppr_from_slabs_kernel(const V* __restrict__ src,
                                                                     V* __restrict__ dst,
                                                                     int64_t n, int k) {
  const int j = threadIdx.x & 63;
  if (j >= k) return;
  const int64_t step = (int64_t)gridDim.x * kPprWaves;
  for (int64_t r = (int64_t)blockIdx.x * kPprWaves + (threadIdx.x >> 6); r < n; r += step)
    dst[r * k + j] = src[ppr_at(r, j, n, k)];
}

hipError_t launch_ppr_from_slabs(int dtype, const void* Xs, void* X, int64_t n, int k,
                                 hipStream_t st) {
  if (n == 0) return hipSuccess;
  const unsigned grid = (unsigned)std::min<int64_t>((n + kPprWaves - 1) / kPprWaves, 8192);
  if (dtype == 0)
    hipLaunchKernelGGL(ppr_from_slabs_kernel<float>, dim3(grid), dim3(kPprThreads), 0, st,
                       static_cast<const float*>(Xs), static_cast<float*>(X), n, k);
  else
    hipLaunchKernelGGL(ppr_from_slabs_kernel<double>, dim3(grid), dim3(kPprThreads), 0, st,
                       static_cast<const double*>(Xs), static_cast<double*>(X), n, k);
  return hipGetLastError();
}

// the caller's row-major X into the slab layout, with X's dangling mass per
// column (the same parts as ppr_dangling_kernel, from the same pass)
template <typename V>
__global__ __launch_bounds__(kPprThreads) void ppr_to_slabs_kernel(
    const V* __restrict__ src, V* __restrict__ dst, const uint32_t* __restrict__ dmask,
    int64_t n, int k, double* __restrict__ part_out) {
  const int j = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  double dsum = 0.0;
  const int64_t step = (int64_t)gridDim.x * kPprWaves * kPprRows;
  for (int64_t r0 = ((int64_t)blockIdx.x * kPprWaves + w) * kPprRows; j < k && r0 < n;
       r0 += step) {
    V v[kPprRows];
#pragma unroll
    for (int u = 0; u < kPprRows; ++u) v[u] = src[min(r0 + u, n - 1) * k + j];
#pragma unroll
    for (int u = 0; u < kPprRows; ++u) {
      const int64_t r = r0 + u;
      if (r < n) {
        dst[ppr_at(r, j, n, k)] = v[u];
        if ((dmask[r >> 5] >> (r & 31)) & 1u) dsum += (double)v[u];
      }
    }
  }
  ppr_block_part(dsum, 0.0, part_out);
}

// sums[2j], sums[2j+1] = totals over the blocks of column j's parts: block j
// of this kernel; thread t adds parts t, t + 256, ... in order, then a
// fixed-order block reduction
__global__ __launch_bounds__(kReduceThreads) void ppr_sum_parts_kernel(
    const double* __restrict__ part, int nblocks, double* __restrict__ sums) {
  const int j = blockIdx.x;
  double d = 0.0, r = 0.0;
  const double2* __restrict__ p2 = reinterpret_cast<const double2*>(part);
  constexpr int kPartILP = 8;  // loads in flight per thread
  for (int b = threadIdx.x; b < nblocks; b += kPartILP * kReduceThreads) {
    double2 v[kPartILP];
#pragma unroll
    for (int u = 0; u < kPartILP; ++u)
      v[u] = p2[(int64_t)min(b + u * kReduceThreads, nblocks - 1) * 64 + j];
#pragma unroll
    for (int u = 0; u < kPartILP; ++u) {
      if (b + u * kReduceThreads < nblocks) {
        d += v[u].x;
        r += v[u].y;
      }
    }
  }
  block_sum2(d, r);
  if (threadIdx.x == 0) {
    sums[2 * j] = d;
    sums[2 * j + 1] = r;
  }
}

int ppr_grid(int64_t n) {
  int64_t g = (n + kPprWaves * kPprRows * 8 - 1) / (kPprWaves * kPprRows * 8);
  if (g > 4096) g = 4096;
  if (g < 1) g = 1;
  return (int)g;
}

// First level for long part lists (the fused SpMM writes one part row per
// block: 54K at R-MAT 22, sigma 5): block g adds rows g, g + G, g + 2G, ...
// with thread t on entry t of a row (rows are read whole, coalesced), in a
// fixed order (eight running sums, then a fixed tree), into row g of out.
constexpr int kPartLevelRows = 1024;  // G; out holds G rows
constexpr int kPartDirectMax = 4096;  // at most this many rows: no first level

__global__ __launch_bounds__(128) void ppr_part_rows_kernel(const double* __restrict__ part,
                                                            int nblocks,
                                                            double* __restrict__ out) {
  const int t = threadIdx.x;
  const int G = gridDim.x;
  double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  int b = blockIdx.x;
  for (; b + 7 * G < nblocks; b += 8 * G) {
#pragma unroll
    for (int u = 0; u < 8; ++u) s[u] += part[((int64_t)b + (int64_t)u * G) * 128 + t];
  }
  for (; b < nblocks; b += G) s[0] += part[(int64_t)b * 128 + t];
  out[(int64_t)blockIdx.x * 128 + t] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

int ppr_sum_scratch_rows() { return kPartLevelRows; }

hipError_t launch_ppr_sum(const double* part, int nblocks, int k, double* sums, double* scratch,
                          hipStream_t st) {
  if (nblocks > kPartDirectMax && scratch != nullptr) {
    hipLaunchKernelGGL(ppr_part_rows_kernel, dim3(kPartLevelRows), dim3(128), 0, st, part,
                       nblocks, scratch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    part = scratch;
    nblocks = kPartLevelRows;
  }
  hipLaunchKernelGGL(ppr_sum_parts_kernel, dim3(k), dim3(kReduceThreads), 0, st, part, nblocks,
                     sums);
  return hipGetLastError();
}

hipError_t launch_ppr_dangling(int dtype, const void* X, const uint32_t* dmask, int64_t n, int k,
                               double* part, double* sums, int grid, hipStream_t st) {
  if (dtype == 0)
    hipLaunchKernelGGL(ppr_dangling_kernel<float>, dim3(grid), dim3(kPprThreads), 0, st,
                       static_cast<const float*>(X), dmask, n, k, part);
  else
    hipLaunchKernelGGL(ppr_dangling_kernel<double>, dim3(grid), dim3(kPprThreads), 0, st,
                       static_cast<const double*>(X), dmask, n, k, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_ppr_sum(part, grid, k, sums, nullptr, st);
}

hipError_t launch_ppr_to_slabs(int dtype, const void* X, void* Xs, const uint32_t* dmask,
                               int64_t n, int k, double* part, double* sums, int grid,
                               hipStream_t st) {
  if (dtype == 0)
    hipLaunchKernelGGL(ppr_to_slabs_kernel<float>, dim3(grid), dim3(kPprThreads), 0, st,
                       static_cast<const float*>(X), static_cast<float*>(Xs), dmask, n, k, part);
  else
    hipLaunchKernelGGL(ppr_to_slabs_kernel<double>, dim3(grid), dim3(kPprThreads), 0, st,
                       static_cast<const double*>(X), static_cast<double*>(Xs), dmask, n, k,
                       part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_ppr_sum(part, grid, k, sums, nullptr, st);
}

hipError_t launch_ppr_fixup(int dtype, const uint32_t* tile_y, int32_t tile_num, void* Y,
                            void* Xn, int64_t n, int k, double alpha, const int32_t* src,
                            const double* sums_in, const uint32_t* dmask, double* part, int grid,
                            hipStream_t st) {
  if (dtype == 0)
    hipLaunchKernelGGL(ppr_fixup_kernel<float>, dim3(grid), dim3(kPprThreads), 0, st, tile_y,
                       tile_num, static_cast<float*>(Y), static_cast<float*>(Xn), n, k, alpha,
                       src, sums_in, dmask, part);
  else
    hipLaunchKernelGGL(ppr_fixup_kernel<double>, dim3(grid), dim3(kPprThreads), 0, st, tile_y,
                       tile_num, static_cast<double*>(Y), static_cast<double*>(Xn), n, k, alpha,
                       src, sums_in, dmask, part);
  return hipGetLastError();
}

hipError_t launch_ppr_resid(int dtype, const void* Xn, const void* Xo, int64_t n, int k,
                            double* part, int grid, hipStream_t st) {
  if (dtype == 0)
    hipLaunchKernelGGL(ppr_resid_kernel<float>, dim3(grid), dim3(kPprThreads), 0, st,
                       static_cast<const float*>(Xn), static_cast<const float*>(Xo), n, k, part);
  else
    hipLaunchKernelGGL(ppr_resid_kernel<double>, dim3(grid), dim3(kPprThreads), 0, st,
                       static_cast<const double*>(Xn), static_cast<const double*>(Xo), n, k,
                       part);
  return hipGetLastError();
}

// ------------------------------------------------ PageRank of many graphs --
//
// The graphs lie on the diagonal of one matrix: graph g owns rows and columns
// [gp[g], gp[g+1]), and its step is the PageRank step of Sec. 5.5.1 with its
// own size, dangling mass and teleport:
//   x'[r] = alpha y[r] + (alpha delta_g + 1 - alpha) / n_g   for r in graph g.
// Rows are cut into chunks of at most kMultiRows rows that never cross a
// graph; chunk c is rows [chunk_row[c], chunk_row[c+1]) of graph
// chunk_graph[c], and graph g's chunks are chunk_ptr[g] .. chunk_ptr[g+1]-1.
// One block per chunk writes the chunk's (dangling mass, l1 change) pair.  A
// graph's pairs are added in chunk order (deterministic) by the next update's
// wavefronts, each for itself, or by a second kernel: after the step whose
// sums the host reads, and after every step where a graph has more than
// kMultiFoldChunks chunks or the update writes hot values (a hot column's
// graph is another than its block's).  Microseconds per iteration with the
// second kernel and without, FP32, 8 edges per row: 64 graphs of 10,000 rows
// 33.8 and 31.8; one graph of 489 chunks 30.2 and 29.0, of 977 49.9 and 49.3,
// of 1,954 77.4 and 79.9 (every wavefront reads all the pairs).

constexpr int kMultiILP = 4;
constexpr int kMultiRows = kReduceThreads * kMultiILP;

int multi_chunk_rows() { return kMultiRows; }

constexpr int kMultiFoldChunks = 512;

// (dangling mass, l1 change) of the chunks c0 .. c1 - 1, in every lane: lane l
// adds chunks c0 + l, c0 + l + 64, ... in order, then a fixed-order wavefront
// reduction
__device__ __forceinline__ double2 multi_graph_sum(const double* __restrict__ part, int c0, int c1,
                                                   int lid) {
  constexpr int kILP = 4;  // loads in flight per lane
  const double2* __restrict__ p2 = reinterpret_cast<const double2*>(part);
  double2 s = {0.0, 0.0};
  for (int c = c0 + lid; c < c1; c += kILP * kOmega) {
    double2 v[kILP];
#pragma unroll
    for (int u = 0; u < kILP; ++u) v[u] = p2[min(c + u * kOmega, c1 - 1)];
#pragma unroll
    for (int u = 0; u < kILP; ++u) {
      if (c + u * kOmega < c1) {
        s.x += v[u].x;
        s.y += v[u].y;
      }
    }
  }
  s.x = wave_sum(s.x);
  s.y = wave_sum(s.y);
  return s;
}

// With hot_n > 0 the kernel also writes the hot-column copy of x' that the
// next SpMV's LDS cache reads: slot s holds column hot_cols[s] of graph
// hot_graph[s], computed with the same operations as that row's x'.
// Without RESID x_old is not read and the l1 parts are 0 (the host reads
// the l1 change only after a chunk's last step).  part_in: the step before's
// pairs, added here instead of read from gsum_in (without hot columns).
template <typename V, bool RESID>
__global__ __launch_bounds__(kReduceThreads) void multi_update_kernel(
    const V* __restrict__ y, const V* __restrict__ x_old, V* __restrict__ x_new,
    const uint32_t* __restrict__ dmask, const int32_t* __restrict__ chunk_row,
    const int32_t* __restrict__ chunk_graph, const int32_t* __restrict__ chunk_ptr,
    const double* __restrict__ gsum_in, const double* __restrict__ part_in,
    const double* __restrict__ gsize, double alpha, double* __restrict__ part_out,
    const int32_t* __restrict__ hot_cols, const int32_t* __restrict__ hot_graph, int32_t hot_n,
    V* __restrict__ x_hot) {
  const int c = blockIdx.x;
  const int64_t r0 = chunk_row[c], r1 = chunk_row[c + 1];
  const int g = chunk_graph[c];
  const V a = (V)alpha;
  V yv[kMultiILP], xo[kMultiILP];
  uint32_t mw[kMultiILP];
#pragma unroll
  for (int u = 0; u < kMultiILP; ++u) {
    const int64_t i = min(r0 + threadIdx.x + (int64_t)u * kReduceThreads, r1 - 1);
    yv[u] = y[i];
    if constexpr (RESID) xo[u] = x_old[i];
    mw[u] = dmask[i >> 5];
  }
  const double delta = part_in != nullptr
                           ? multi_graph_sum(part_in, chunk_ptr[g], chunk_ptr[g + 1],
                                             threadIdx.x & (kOmega - 1)).x
                           : gsum_in[2 * g];
  const V tele = (V)((alpha * delta + 1.0 - alpha) / gsize[g]);
  double dsum = 0.0, rsum = 0.0;
#pragma unroll
  for (int u = 0; u < kMultiILP; ++u) {
    const int64_t i = r0 + threadIdx.x + (int64_t)u * kReduceThreads;
    if (i < r1) {
      const V xn = fma(a, yv[u], tele);
      x_new[i] = xn;
      if constexpr (RESID) rsum += fabs((double)xn - (double)xo[u]);
      if ((mw[u] >> (i & 31)) & 1u) dsum += (double)xn;
    }
  }
  for (int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; h < hot_n;
       h += (int64_t)gridDim.x * blockDim.x) {
    const int gh = hot_graph[h];
    const V th = (V)((alpha * gsum_in[2 * gh] + 1.0 - alpha) / gsize[gh]);
    x_hot[h] = fma(a, y[hot_cols[h]], th);
  }
  block_sum2(dsum, rsum);
  if (threadIdx.x == 0) {
    part_out[2 * c] = dsum;
    part_out[2 * c + 1] = rsum;
  }
}

template <typename V>
__global__ __launch_bounds__(kReduceThreads) void multi_dangling_kernel(
    const V* __restrict__ x, const uint32_t* __restrict__ dmask,
    const int32_t* __restrict__ chunk_row, double* __restrict__ part_out) {
  const int c = blockIdx.x;
  const int64_t r0 = chunk_row[c], r1 = chunk_row[c + 1];
  double dsum = 0.0, zero = 0.0;
  for (int64_t i = r0 + threadIdx.x; i < r1; i += kReduceThreads)
    if ((dmask[i >> 5] >> (i & 31)) & 1u) dsum += (double)x[i];
  block_sum2(dsum, zero);
  if (threadIdx.x == 0) {
    part_out[2 * c] = dsum;
    part_out[2 * c + 1] = 0.0;
  }
}

// one wavefront per graph
__global__ __launch_bounds__(256) void multi_sum_kernel(const double* __restrict__ part,
                                                         const int32_t* __restrict__ chunk_ptr,
                                                         int n_graphs,
                                                         double* __restrict__ gsum_out) {
  const int g = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lid = threadIdx.x & 63;
  if (g >= n_graphs) return;
  const double2 s = multi_graph_sum(part, chunk_ptr[g], chunk_ptr[g + 1], lid);
  if (lid == 0) {
    gsum_out[2 * g] = s.x;
    gsum_out[2 * g + 1] = s.y;
  }
}

static hipError_t launch_multi_sum(const double* part, const int32_t* chunk_ptr, int n_graphs,
                                   double* gsum_out, hipStream_t st) {
  hipLaunchKernelGGL(multi_sum_kernel, dim3((unsigned)((n_graphs + 3) / 4)), dim3(256), 0, st,
                     part, chunk_ptr, n_graphs, gsum_out);
  return hipGetLastError();
}

hipError_t launch_multi_dangling(int dtype, const void* x, const uint32_t* dmask,
                                 const MultiTables& mt, double* gsum_out, hipStream_t st) {
  if (dtype == 0)
    hipLaunchKernelGGL(multi_dangling_kernel<float>, dim3((unsigned)mt.n_chunks),
                       dim3(kReduceThreads), 0, st, static_cast<const float*>(x), dmask,
                       mt.chunk_row, mt.part[0]);
  else
    hipLaunchKernelGGL(multi_dangling_kernel<double>, dim3((unsigned)mt.n_chunks),
                       dim3(kReduceThreads), 0, st, static_cast<const double*>(x), dmask,
                       mt.chunk_row, mt.part[0]);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_multi_sum(mt.part[0], mt.chunk_ptr, mt.n_graphs, gsum_out, st);
}

template <typename V>
static void multi_update_launch(bool resid, const void* y, const void* x_old, void* x_new,
                                const uint32_t* dmask, const MultiTables& mt, double alpha,
                                int cur, const double* gsum_in, bool fold, hipStream_t st,
                                const int32_t* hot_cols, int32_t hot_n, void* x_hot) {
  const double* part_in = fold ? mt.part[cur] : nullptr;
  double* part_out = mt.part[cur ^ 1];
  const V* yv = static_cast<const V*>(y);
  const V* xo = static_cast<const V*>(x_old);
  V* xn = static_cast<V*>(x_new);
  V* xh = static_cast<V*>(x_hot);
  if (resid)
    hipLaunchKernelGGL((multi_update_kernel<V, true>), dim3((unsigned)mt.n_chunks),
                       dim3(kReduceThreads), 0, st, yv, xo, xn, dmask, mt.chunk_row,
                       mt.chunk_graph, mt.chunk_ptr, gsum_in, part_in, mt.gsize, alpha, part_out,
                       hot_cols, mt.hot_graph, hot_n, xh);
  else
    hipLaunchKernelGGL((multi_update_kernel<V, false>), dim3((unsigned)mt.n_chunks),
                       dim3(kReduceThreads), 0, st, yv, xo, xn, dmask, mt.chunk_row,
                       mt.chunk_graph, mt.chunk_ptr, gsum_in, part_in, mt.gsize, alpha, part_out,
                       hot_cols, mt.hot_graph, hot_n, xh);
}

hipError_t launch_multi_update(int dtype, const void* y, const void* x_old, void* x_new,
                               const uint32_t* dmask, const MultiTables& mt, double alpha,
                               int cur, const double* gsum_in, double* gsum_out,
                               hipStream_t st, const int32_t* hot_cols, int32_t hot_n,
                               void* x_hot, bool resid) {
  if (hot_n > 0 && mt.hot_graph == nullptr) return hipErrorInvalidValue;
  const bool fold = hot_n == 0 && mt.max_chunks <= kMultiFoldChunks;
  if (dtype == 0)
    multi_update_launch<float>(resid, y, x_old, x_new, dmask, mt, alpha, cur, gsum_in, fold, st,
                               hot_cols, hot_n, x_hot);
  else
    multi_update_launch<double>(resid, y, x_old, x_new, dmask, mt, alpha, cur, gsum_in, fold, st,
                                hot_cols, hot_n, x_hot);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || (fold && !resid)) return e;
  return launch_multi_sum(mt.part[cur ^ 1], mt.chunk_ptr, mt.n_graphs, gsum_out, st);
}

}  // namespace merbit
