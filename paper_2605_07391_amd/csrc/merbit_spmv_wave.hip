// MERBIT SpMV with one commit unit per tile (b = 64 lanes = one wavefront),
// persistent and software pipelined, for gfx950.
//
// Same method as the block kernel (Sec. 4.2 of the MERBIT paper): tiles of 64
// lanes x sigma merge-path steps, coalesced loads of values / col_ind, products
// staged in LDS, each lane walking its descriptor, a head-flagged segmented
// scan across the wavefront, long-row fast tiles and empty-tile skips.  The
// paper's block size b is set to one wavefront, so wavefronts never wait for
// each other:
//   - rows that start and end inside a tile are complete after the tile's own
//     scan and are stored with coalesced writes from the wavefront's LDS slots;
//   - a short row (at most kOwnRowMax nonzeros) that begins before the tile is
//     finished by the tile it ends in, which adds up the few nonzeros before it
//     again, and is stored like the others;
//   - a long row that crosses tiles is added to y atomically by each of them; y
//     is zero at every tile's first row before the launch (dual buffer: each
//     tile zeroes z at its first row, Sec. 4.2 opt. (3)).
// A block of WAVES wavefronts is resident for the whole launch.  The tiles
// (with the tiles split into ranges, those of the block's range) are dealt
// round robin over the blocks (singly, or in runs in a large FP64 plan), and a block's wavefronts take the block's tiles
// one at a time from a counter in LDS.  The loads of the next tile (bounds,
// descriptor, col_ind, values) are issued before the current tile's gathers
// are consumed, so that the two wait together (they lie under branches, so the
// compiler waits for all of them before the walk).
//
// What bounds it: the x gathers (L1 misses in flight per CU times the latency
// of L2) and, below about 10M nonzeros, the fixed costs (the copy of the hot
// values, the launch).  Time per tile varies by its columns, and neighbouring
// tiles are alike, so wavefronts with a fixed sequence of tiles (g, g + W,
// ...: 16 neighbours per block) ended 30-68 us into a 68 us launch on R-MAT 20
// FP32 (mean 48).  Dealing single tiles over the blocks and taking them from
// the block's counter: 39-56 us.  With the walk below, per SpMV: R-MAT 20 70.2
// -> 60.2 us (FP32), 97.7 -> 90 us (FP64), Chung-Lu 700,001 45.3 -> 38.7 us
// (FP32), R-MAT 22 on 8 stripes, 64-bit descriptors, sigma 28, 210 -> 196 us
// (FP32; there it replaces one global counter per range, which cost an atomic
// round trip per tile).  Deals of 2 or 4 tiles at a time were 1 and 2 %
// slower; a software pipeline that issues the next tile's gathers before the
// current walk, and gathers split from the LDS reads (buffer loads, or loads
// under a branch, where the compiler now merges both into one flat load) made
// no difference.  Short rows that cross tiles finished by one tile, with no
// atomics (an atomic pair per tile) and, where no row is long, no launch that
// zeroes y first: Chung-Lu 700,001 FP64 53.5 -> 45 us, 1,000,000 vertices of
// degree 80 FP64 392 -> 346 us, 10,000 vertices FP32 10.6 -> 7.5 us.
//
// HOT: the block first copies the hot x values into LDS (the plan's recoded
// column stream marks hot columns as -1 - slot) and serves those gathers from
// LDS.
#include "merbit_internal.hpp"

namespace merbit {

// D: the descriptor word, uint32_t (sigma <= 12) or uint64_t (sigma <= 40)
template <typename V, int SIGMA, typename D>
struct WaveTile {
  int x_ws;
  int x_se;
  uint32_t tyw;
  int y_we;
  D desc;
  int cc[SIGMA];
  V vv[SIGMA];
  // first nonzero of the tile's first row (-1: a long row) and whether the
  // row it ends in is short; the part of a short first row that lies before
  // the tile is x_ws - hd nonzeros, lane l holding the l-th
  int hd;
  bool last_short;
  int pc;
  V pv;
};

template <typename D>
__device__ __forceinline__ D load_desc(const SpmvArgs& a, int j);
template <>
__device__ __forceinline__ uint32_t load_desc<uint32_t>(const SpmvArgs& a, int j) {
  return a.lane_desc[j];
}
template <>
__device__ __forceinline__ uint64_t load_desc<uint64_t>(const SpmvArgs& a, int j) {
  return a.lane_desc64[j];
}

// Buffer-resource loads of the tile stream: faster for FP32 (both descriptor
// widths) and for FP64 with 64-bit descriptors (3.7-5 % per SpMV on R-MAT 22),
// slower by 2 % for FP64 with 32-bit descriptors, which keeps plain loads.
template <typename V, typename D>
constexpr bool kBufferStream = sizeof(V) == 4 || sizeof(D) == 8;
// How a gather picks LDS (hot columns) or memory: one flat load from a selected
// address, or a load from memory for every lane (hot ones repeat x[0]) and one
// from LDS.  The flat load is faster (sigma 28 FP32 on R-MAT 22: 199 against
// 203 us per SpMV; FP64 sigma 24 306 against 322, sigma 14 300 against 312, on
// R-MAT 20 75 against 77) but for FP64 with 64-bit descriptors of sigma 16 (306
// against 285 us).  Written as a branch, the compiler emits the flat load in
// some instances and in others a global and an LDS load into one register, each
// waiting for the one before (sigma 16 FP32: 297 against 213 us).
template <typename V, int SIGMA, typename D>
constexpr bool kFlatGather = sizeof(V) == 4 || sizeof(D) == 4 || SIGMA != 16;

// word 3 of a raw (unformatted, stride 0) buffer resource on gfx950
constexpr int kBufferWord3 = 0x00020000;
// cache policy bits of a gfx950 buffer load: nt (streaming, evicted first)
constexpr int kPolicyStream = 2;
// hot x values loaded per lane before they are stored to LDS (128 bytes:
// 16 -> 32 took FP32 sigma 28 from 226 to 224 us per SpMV; 64 FP64 values
// spill in the 1,024-lane kernels)
template <typename V>
constexpr int kHotBatch = 128 / (int)sizeof(V);

// A load through the constant address space: the tile bounds are never
// written during a launch, and with atomics in the loop the compiler could
// otherwise not prove that, and would load the (uniform) bounds with vector
// loads that wait for every gather in flight.
template <typename T>
__device__ __forceinline__ T const_load(const T* p, int i) {
  typedef const __attribute__((address_space(4))) T ConstT;
  return ((ConstT*)p)[i];
}

template <typename V, int SIGMA, typename D>
__device__ __forceinline__ void wave_load_tile(const SpmvArgs& a, const int32_t* __restrict__ col,
                                               const V* __restrict__ val, int t, int lid,
                                               WaveTile<V, SIGMA, D>& s) {
  s.x_ws = const_load(a.tile_x, t);
  s.x_se = const_load(a.tile_x, t + 1) - s.x_ws;
  s.tyw = const_load(a.tile_y, t);
  s.y_we = (int)(const_load(a.tile_y, t + 1) & kRowMask);
  s.hd = const_load(a.row_start, t);
  s.last_short = const_load(a.row_start, t + 1) >= 0;
  s.pc = 0;
  s.pv = V(0);
  if (s.hd >= 0 && lid < s.x_ws - s.hd) {
    s.pc = col[s.hd + lid];
    s.pv = val[s.hd + lid];
  }
  const bool normal = s.x_se > 0 && !(s.tyw & kFastBit);
  s.desc = 0;
  if (normal) s.desc = load_desc<D>(a, min(t * kOmega + lid, a.lane_num - 1));
  // A tile without nonzeros reads nothing: col / val may be empty (nnz = 0).
  // The branch is uniform across the wavefront.
  if (s.x_se > 0) {
    if constexpr (kBufferStream<V, D>) {
      // buffer loads over the tile's own range (streaming policy): one 32-bit
      // offset per lane instead of a 64-bit address per load, and reads past
      // the tile's end return 0 without a clamp.  A zero column gathers x[0]
      // (x is not empty when the tile has nonzeros) and its product is never
      // staged.
      const int xws = __builtin_amdgcn_readfirstlane(s.x_ws);
      const int xse = __builtin_amdgcn_readfirstlane(s.x_se);
      const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(col + xws), (short)0, xse * 4, kBufferWord3);
      const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(val + xws), (short)0, xse * (int)sizeof(V), kBufferWord3);
#pragma unroll
      for (int it = 0; it < SIGMA; ++it) {
        const int k = lid + it * kOmega;
        s.cc[it] = (int)__builtin_amdgcn_raw_buffer_load_b32(rc, k * 4, 0, kPolicyStream);
        if constexpr (sizeof(V) == 4)
          s.vv[it] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(rv, k * 4, 0,
                                                                                kPolicyStream));
        else
          s.vv[it] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(rv, k * 8, 0,
                                                                                kPolicyStream));
      }
    } else {
#pragma unroll
      for (int it = 0; it < SIGMA; ++it) {
        const int k = min(lid + it * kOmega, s.x_se - 1);
        s.cc[it] = __builtin_nontemporal_load(col + s.x_ws + k);
        s.vv[it] = __builtin_nontemporal_load(val + s.x_ws + k);
      }
    }
  } else {
#pragma unroll
    for (int it = 0; it < SIGMA; ++it) {
      s.cc[it] = 0;
      s.vv[it] = V(0);
    }
  }
}

// Steps of the walk whose products are read from LDS together.  4 is the best
// or level with it everywhere (R-MAT 20 / 22, sigma 7-28); more cost
// registers: FP64 sigma 20 on R-MAT 22 took 291 / 302 / 309 us per SpMV at 4 /
// 8 / 20 steps.
constexpr int kWalkGroup = 4;

// The kernel's descriptor argument: the word, or InRuns of it where the tiles
// are dealt in runs of WAVES neighbours (SpmvArgs::runs).
template <typename D>
struct InRuns {};
template <typename DESC>
struct DescOf {
  typedef DESC word;
  static constexpr bool runs = false;
};
template <typename D>
struct DescOf<InRuns<D>> {
  typedef D word;
  static constexpr bool runs = true;
};

template <typename V, int SIGMA, int WAVES, bool HOT, typename DESC>
__global__ __launch_bounds__(WAVES * 64) void spmv_wave_kernel(SpmvArgs a) {
  typedef typename DescOf<DESC>::word D;
  constexpr bool RUNS = DescOf<DESC>::runs;
  constexpr int BITS = ceil_log2(kOmega * SIGMA);
  constexpr uint32_t FMASK = (1u << BITS) - 1u;
  static_assert(2 * BITS + SIGMA <= 8 * (int)sizeof(D), "descriptor does not fit");
  constexpr int WLDS = kOmega * SIGMA;  // per wavefront: products, then inner-row slots
  __shared__ V s_stage[WAVES * WLDS];
  __shared__ int s_next;  // the block's next tile (its place in the block's sequence)

  const int32_t* __restrict__ col = a.col;
  const V* __restrict__ val = static_cast<const V*>(a.val);
  const V* __restrict__ x = static_cast<const V*>(a.x);
  V* __restrict__ y = static_cast<V*>(a.y);
  V* __restrict__ z = static_cast<V*>(a.z);

  const int tid = threadIdx.x;
  const int lid = tid & (kOmega - 1);
  const int wid = __builtin_amdgcn_readfirstlane(tid / kOmega);
  V* s_w = s_stage + wid * WLDS;

  // this block's part of the tiles and of the hot values (one part unless
  // the plan splits the tiles into ranges)
  int t_begin = 0, t_end = a.tile_num, slot = blockIdx.x, slots = a.grid;
  int h_begin = 0, h_num = a.hot_n;
  if (a.ranges > 1) {
    const int k = blockIdx.x % a.ranges;
    t_begin = a.range_tile[k];
    t_end = a.range_tile[k + 1];
    slot = blockIdx.x / a.ranges;
    slots = a.grid / a.ranges;
    if (HOT) {
      h_begin = a.hot_off[k];
      h_num = a.hot_off[k + 1] - h_begin;
    }
  }

  if (tid == 0) s_next = WAVES;
  extern __shared__ __align__(16) unsigned char s_dyn[];
  const V* s_hot = reinterpret_cast<const V*>(s_dyn);
  if (HOT) {
    // kHotBatch loads per lane in flight before their LDS stores: the copy
    // takes h_num / (kHotBatch * block lanes) memory round trips, not
    // h_num / block lanes (one block per CU waits for it)
    // (buffer loads over the block's hot slice: reads past its end return 0)
    constexpr int NT = WAVES * kOmega;
    V* dst = reinterpret_cast<V*>(s_dyn);
    const __amdgpu_buffer_rsrc_t rh = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(static_cast<const V*>(a.x_hot) + h_begin), (short)0, h_num * (int)sizeof(V),
        kBufferWord3);
    for (int s0 = tid; s0 < h_num; s0 += kHotBatch<V> * NT) {
      V hv[kHotBatch<V>];
#pragma unroll
      for (int u = 0; u < kHotBatch<V>; ++u) {
        const int off = (s0 + u * NT) * (int)sizeof(V);
        if constexpr (sizeof(V) == 4)
          hv[u] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(rh, off, 0, 0));
        else
          hv[u] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(rh, off, 0, 0));
      }
#pragma unroll
      for (int u = 0; u < kHotBatch<V>; ++u) {
        const int s = s0 + u * NT;
        if (s < h_num) dst[s] = hv[u];
      }
    }
  }
  __syncthreads();

  // The range's tiles are dealt round robin over its blocks, and the block's
  // wavefronts take the block's tiles one at a time from a counter in LDS, so
  // a wavefront that meets cheap tiles takes more of them.
  auto take = [&]() -> int {
    int q = 0;
    if (lid == 0) q = atomicAdd(&s_next, 1);
    return q;
  };
  auto tile_at = [&](int i) -> int {
    i = __builtin_amdgcn_readfirstlane(i);
    const int tile = RUNS ? t_begin + (i / WAVES * slots + slot) * WAVES + i % WAVES
                          : t_begin + i * slots + slot;
    return tile < t_end ? tile : t_end;
  };
  // x of column c, or for a hot column (kFlatGather off) an x value that x_of
  // replaces by the one in LDS
  auto gather = [&](int c) -> V {
    if constexpr (HOT && kFlatGather<V, SIGMA, D>) {
      const V* p = c < 0 ? s_hot + (-1 - c) : x + c;
      return *p;
    }
    return x[HOT ? max(c, 0) : c];
  };
  auto x_of = [&](int c, V g) -> V {
    if constexpr (HOT && !kFlatGather<V, SIGMA, D>) {
      const V h = s_hot[c < 0 ? -1 - c : 0];
      return c < 0 ? h : g;
    }
    return g;
  };
  int t = tile_at(wid);
  int tn = t_end;
  WaveTile<V, SIGMA, D> cur;
  if (t < t_end) {
    wave_load_tile<V, SIGMA, D>(a, col, val, t, lid, cur);
    tn = tile_at(take());
  }
  while (t < t_end) {
    // gathers of the current tile (none for a tile without nonzeros: x may be
    // empty then)
    V g[SIGMA];
    if (cur.x_se > 0) {
#pragma unroll
      for (int it = 0; it < SIGMA; ++it) {
        g[it] = gather(cur.cc[it]);
      }
    }
    // (x is not empty if the first row has nonzeros before the tile)
    const int before = cur.hd >= 0 ? cur.x_ws - cur.hd : 0;
    V pg = V(0);
    if (before > 0) pg = gather(cur.pc);
    // the tile after next, then the loads of the next tile: both go out
    // before the gathers are consumed
    int q = 0;
    if (tn < t_end) q = take();
    WaveTile<V, SIGMA, D> nxt;
    if (tn < t_end) wave_load_tile<V, SIGMA, D>(a, col, val, tn, lid, nxt);

    const int x_se = cur.x_se;
    const int y_ws = (int)(cur.tyw & kRowMask);
    const int y_we = cur.y_we;
    const bool last_short = cur.last_short;
    const bool own = cur.hd >= 0;  // this tile finishes its first row by itself
    V pre = V(0);
    if (before > 0) {
      pre = cur.pv * x_of(cur.pc, pg);  // lanes past `before` hold a zero value and a gather of x[0]
      if (lid >= before) pre = V(0);
      for (int k = kOmega + lid; k < before; k += kOmega)
        pre += val[cur.hd + k] * x_of(col[cur.hd + k], gather(col[cur.hd + k]));
      pre = wave_total(pre);
    }
    if (x_se == 0) {
      // down steps only: the rows strictly inside the tile are empty
      for (int r = y_ws + 1 + lid; r < y_we; r += kOmega) y[r] = V(0);
      if (own && lid == 0 && y_we > y_ws) y[y_ws] = pre;
    } else if (cur.tyw & kFastBit) {
      // single-row tile (Sec. 4.2 opt. (1))
      V acc = V(0);
#pragma unroll
      for (int it = 0; it < SIGMA; ++it)
        if (lid + it * kOmega < x_se) acc += cur.vv[it] * x_of(cur.cc[it], g[it]);
      acc = wave_total(acc);
      if (lid == 0 && !own) global_add(&y[y_ws], acc);
    } else {
      wave_lds_sync();  // the previous tile's commit has read its slots
#pragma unroll
      for (int it = 0; it < SIGMA; ++it) {
        const int k = lid + it * kOmega;
        if (k < x_se) s_w[k] = cur.vv[it] * x_of(cur.cc[it], g[it]);
      }
      wave_lds_sync();
      // walk (Algorithm tile_normal_tackle): the row that ends at a down step
      // is written to slot x_se + (its index in the tile), which no other lane
      // writes.  A lane's right steps read consecutive products, so with xo
      // the next product and C = x_off + y_off of the lane, step k's product
      // is s_w[xo] and its row's slot x_se + C + k - xo: neither needs a
      // product's value, so the reads of a group of steps go out together (one
      // read at a time, each waited for before the next step, took 4,200 cycles
      // per tile at sigma 12 against 3,300).
      const int j = t * kOmega + lid;
      V sum = V(0);
      const int start_off = (int)((cur.desc >> BITS) & FMASK);
      const D flags = cur.desc >> (2 * BITS);
      bool has_down = flags != 0;
      int xo = (int)(cur.desc & FMASK);
      const int sb = x_se + xo + start_off;
      if (t < a.tile_num - 1) {
#pragma unroll
        for (int k0 = 0; k0 < SIGMA; k0 += kWalkGroup) {
          V v[kWalkGroup];
          int at[kWalkGroup];
#pragma unroll
          for (int u = 0; u < kWalkGroup; ++u) {
            const int k = k0 + u;
            if (k < SIGMA) {
              at[u] = xo;
              v[u] = s_w[xo];
              xo += (int)((~flags >> k) & 1);
            }
          }
#pragma unroll
          for (int u = 0; u < kWalkGroup; ++u) {
            const int k = k0 + u;
            if (k < SIGMA) {
              const bool down = (flags >> k) & 1;
              if (down) s_w[sb + k - at[u]] = sum;
              sum = down ? V(0) : sum + v[u];
            }
          }
        }
      } else {
        // the last tile: lanes past the path take no step
        has_down = has_down && j < a.lane_num;
        const int steps = min(SIGMA, a.path_len - j * SIGMA);
#pragma unroll 1
        for (int k = 0; k < steps; ++k) {
          if ((flags >> k) & 1) {
            s_w[sb + k - xo] = sum;
            sum = V(0);
          } else {
            sum += s_w[xo++];
          }
        }
      }
      const unsigned long long heads = __ballot(has_down) | 1ull;
      const unsigned long long upto = lid == kOmega - 1 ? ~0ull : ((2ull << lid) - 1ull);
      const int seg = 63 - __builtin_clzll(heads & upto);
      const V scan = wave_segmented_scan(sum, lid, seg);
      const V carry = dpp_move<kWaveShr1, 0xF>(scan);
      if (has_down) {
        // the first row that ends in this lane may begin in lanes before it
        V* slot = s_w + x_se + start_off;
        const V row_val = *slot + (lid > 0 ? carry : V(0));
        if (start_off != 0) *slot = row_val;       // begun inside the tile
        else if (own) y[y_ws] = pre + row_val;     // the tile's first row
        else global_add(&y[y_ws], row_val);
      }
      // the last segment belongs to the row the tile ends in
      if (lid == kOmega - 1 && !last_short && y_we < a.n_rows && scan != V(0))
        global_add(&y[y_we], scan);
      wave_lds_sync();
      for (int r = lid + 1; r < y_we - y_ws; r += kOmega) y[y_ws + r] = s_w[x_se + r];
    }
    if (z != nullptr && lid == 0) z[y_ws] = V(0);
    if (tn >= t_end) break;
    cur = nxt;
    t = tn;
    tn = tile_at(q);
  }
}

// kernels that exist with runs: instances of their own, as the choice at run
// time cost plans that deal single tiles (FP64 Chung-Lu 700,001 46.2 -> 46.4 us)
template <typename V, int W, bool H, typename D>
constexpr bool kHasRuns = sizeof(V) == 8 && sizeof(D) == 4 && H && W >= kRunsMinWaves;

template <typename V, int S, int W, bool H, typename D>
static hipError_t launch_wave_t(const SpmvArgs& a, size_t dyn, hipStream_t st) {
  if constexpr (kHasRuns<V, W, H, D>) {
    if (a.runs) {
      hipLaunchKernelGGL((spmv_wave_kernel<V, S, W, H, InRuns<D>>), dim3((unsigned)a.grid),
                         dim3(W * kOmega), dyn, st, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((spmv_wave_kernel<V, S, W, H, D>), dim3((unsigned)a.grid), dim3(W * kOmega),
                     dyn, st, a);
  return hipGetLastError();
}

template <typename V, int S, int W, bool H, typename D>
static hipError_t set_wave_lds_t(size_t bytes) {
  static std::mutex mu;
  static size_t granted[kMaxLdsDevices] = {};
  const hipError_t e = raise_dynamic_lds(
      reinterpret_cast<const void*>(&spmv_wave_kernel<V, S, W, H, D>), bytes, mu, granted);
  if constexpr (kHasRuns<V, W, H, D>) {
    static std::mutex mu_runs;
    static size_t granted_runs[kMaxLdsDevices] = {};
    if (e == hipSuccess)
      return raise_dynamic_lds(
          reinterpret_cast<const void*>(&spmv_wave_kernel<V, S, W, H, InRuns<D>>), bytes, mu_runs,
          granted_runs);
  }
  return e;
}

// resident blocks per CU without dynamic LDS
template <typename V, int S, int W, bool H, typename D>
static hipError_t wave_resident_t(int* blocks) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(
      blocks, reinterpret_cast<const void*>(&spmv_wave_kernel<V, S, W, H, D>), W * kOmega, 0);
}

struct WaveEntry {
  hipError_t (*launch)(const SpmvArgs&, size_t, hipStream_t);
  hipError_t (*set_lds)(size_t);
  hipError_t (*resident)(int*);
};

#define MERBIT_WCASE(S, D) \
  case S: return WaveEntry{launch_wave_t<V, S, W, H, D>, set_wave_lds_t<V, S, W, H, D>, \
                           wave_resident_t<V, S, W, H, D>};

template <typename V, int W, bool H>
static WaveEntry wave_pick_sigma(int sigma) {
  switch (sigma) {
    MERBIT_WCASE(1, uint32_t) MERBIT_WCASE(2, uint32_t) MERBIT_WCASE(3, uint32_t)
    MERBIT_WCASE(4, uint32_t) MERBIT_WCASE(5, uint32_t) MERBIT_WCASE(6, uint32_t)
    MERBIT_WCASE(7, uint32_t) MERBIT_WCASE(8, uint32_t) MERBIT_WCASE(9, uint32_t)
    MERBIT_WCASE(10, uint32_t) MERBIT_WCASE(11, uint32_t) MERBIT_WCASE(12, uint32_t)
    default: return WaveEntry{nullptr, nullptr, nullptr};
  }
}

// 64-bit descriptors: longer lanes than 32 bits allow.  FP32: sigma 16, 20,
// 24, 28, 32; FP64 (twice the registers per value): sigma 14, 16, 20, 24.  256 or
// 512 lanes.
template <typename V, int W, bool H>
static WaveEntry wave_pick_sigma64(int sigma) {
  if constexpr (sizeof(V) == 4) {
    switch (sigma) {
      MERBIT_WCASE(16, uint64_t) MERBIT_WCASE(20, uint64_t) MERBIT_WCASE(24, uint64_t)
      MERBIT_WCASE(28, uint64_t) MERBIT_WCASE(32, uint64_t)
      default: return WaveEntry{nullptr, nullptr, nullptr};
    }
  } else {
    switch (sigma) {
      MERBIT_WCASE(14, uint64_t) MERBIT_WCASE(16, uint64_t) MERBIT_WCASE(20, uint64_t)
      MERBIT_WCASE(24, uint64_t)
      default: return WaveEntry{nullptr, nullptr, nullptr};
    }
  }
}
#undef MERBIT_WCASE

template <typename V, bool H>
static WaveEntry wave_pick_waves(int sigma, int waves, bool desc64) {
  if (desc64) {
    switch (waves) {
      case 4: return wave_pick_sigma64<V, 4, H>(sigma);
      case 8: return wave_pick_sigma64<V, 8, H>(sigma);
      default: return WaveEntry{nullptr, nullptr, nullptr};
    }
  }
  switch (waves) {
    case 4: return wave_pick_sigma<V, 4, H>(sigma);
    case 8: return wave_pick_sigma<V, 8, H>(sigma);
    case 16: return wave_pick_sigma<V, 16, H>(sigma);
    default: return WaveEntry{nullptr, nullptr, nullptr};
  }
}

static WaveEntry wave_pick(int dtype, int sigma, int waves, bool hot, bool desc64) {
  if (dtype == 0) return hot ? wave_pick_waves<float, true>(sigma, waves, desc64)
                             : wave_pick_waves<float, false>(sigma, waves, desc64);
  if (dtype == 1) return hot ? wave_pick_waves<double, true>(sigma, waves, desc64)
                             : wave_pick_waves<double, false>(sigma, waves, desc64);
  return WaveEntry{nullptr, nullptr, nullptr};
}

bool spmv_wave_supported(int dtype, int sigma, int waves, bool hot, bool desc64) {
  return wave_pick(dtype, sigma, waves, hot, desc64).launch != nullptr;
}

hipError_t launch_spmv_wave(int dtype, int sigma, int waves, bool hot, size_t hot_lds_bytes,
                            const SpmvArgs& a, hipStream_t st, bool desc64) {
  WaveEntry k = wave_pick(dtype, sigma, waves, hot, desc64);
  if (!k.launch) return hipErrorInvalidValue;
  return k.launch(a, hot ? hot_lds_bytes : 0, st);
}

hipError_t spmv_wave_resident(int dtype, int sigma, int waves, bool desc64, int* blocks) {
  WaveEntry k = wave_pick(dtype, sigma, waves, false, desc64);
  if (!k.resident) return hipErrorInvalidValue;
  return k.resident(blocks);
}

hipError_t spmv_wave_set_hot_lds(int dtype, int sigma, int waves, size_t bytes, bool desc64) {
  WaveEntry k = wave_pick(dtype, sigma, waves, true, desc64);
  if (!k.set_lds) return hipErrorInvalidValue;
  return k.set_lds(bytes);
}

}  // namespace merbit
