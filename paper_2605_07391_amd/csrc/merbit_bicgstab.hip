// Vector kernels of BiCGSTAB (van der Vorst 1992), the second iterative
// workload of Sec. 5.5.2, around the plan's fused SpMV.  Iteration i:
//   update_p : rho_i = (r^, r_i); beta = (rho_i / rho_{i-1}) (alpha_{i-1} / omega_{i-1});
//              p = r + beta (p - omega_{i-1} v)          (p = r at i = 0)
//   SpMV     : v = A p
//   dot1     : (r^, v)
//   update_s : alpha_i = rho_i / (r^, v);  s = r - alpha_i v
//   SpMV     : t = A s
//   dot2     : (t, s), (t, t)
//   update_xr: omega_i = (t, s) / (t, t);  x += alpha_i p + omega_i s;
//              r = s - omega_i t;  (r^, r), (r, r) for the next iteration
// Every dot product is reduced per block into a (first, second) pair of
// doubles; each consumer kernel sums the pairs itself in block order, so the
// scalars are bit-identical in every block and across runs, and no scalar
// crosses a kernel boundary through a device-scope fence.  The pair arrays of
// consecutive iterations alternate, so iteration i still sees i - 1's.
// Divisions by zero are guarded (the quotient is taken as 0): omega = 0 when
// t = 0 (s = 0, x + alpha p is exact), alpha = 0 when (r^, v) = 0 and
// beta = 0 when rho_{i-1} or omega_{i-1} is 0; the host reports a breakdown
// when rho reaches 0 before convergence.
#include "merbit_internal.hpp"

namespace merbit {

// What bounds these kernels: few blocks with a chain of memory round trips
// each (n = 1M: 256 blocks, 16 elements per thread).  So every pass has
// kBicgILP elements per thread in flight, and the pair arrays that a kernel
// needs are loaded and reduced together.  One element and one array at a time,
// R-MAT 20 FP64 took 11.1 / 7.0 / 8.6 / 6.5 / 12.6 us for update_p / dot1 /
// update_s / dot2 / update_xr; now 9.4 / 4.7 / 7.2 / 4.7 / 12.1 us,
// the updates of p and s with the hot values of the next SpMV (a gather of its
// own took 4.6 us each).
constexpr int kBicgILP = 4;

// Totals of both components of N arrays of G pairs each, identical in every
// block and added in the same order whatever N is.
template <int N>
__device__ __forceinline__ void sum_pairs(const double* const (&part)[N], int G,
                                          double (&tot)[2 * N]) {
  constexpr int W = kReduceThreads / kOmega;
  __shared__ double s_w[W][2 * N];
  double t[2 * N];
#pragma unroll
  for (int q = 0; q < 2 * N; ++q) t[q] = 0.0;
  for (int k = threadIdx.x; k < G; k += kReduceThreads) {
#pragma unroll
    for (int q = 0; q < N; ++q) {
      t[2 * q] += part[q][2 * k];
      t[2 * q + 1] += part[q][2 * k + 1];
    }
  }
#pragma unroll
  for (int q = 0; q < 2 * N; ++q) t[q] = wave_sum(t[q]);
  if ((threadIdx.x & (kOmega - 1)) == 0) {
#pragma unroll
    for (int q = 0; q < 2 * N; ++q) s_w[threadIdx.x / kOmega][q] = t[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2 * N; ++q) {
    tot[q] = 0.0;
    for (int w = 0; w < W; ++w) tot[q] += s_w[w][q];
  }
}

__device__ __forceinline__ double safe_div(double a, double b) { return b != 0.0 ? a / b : 0.0; }

__device__ __forceinline__ void write_pair(double* part, double a, double b) {
  block_sum2(a, b);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = a;
    part[2 * blockIdx.x + 1] = b;
  }
}

// passes over the vectors: thread t of a block takes elements base, base +
// kReduceThreads, ... (kBicgILP of them); BICG_AT clamps, BICG_ON tests
#define BICG_PASS(base)                                                                     \
  for (int64_t base = (int64_t)blockIdx.x * kReduceThreads * kBicgILP + threadIdx.x; base < n; \
       base += (int64_t)gridDim.x * kReduceThreads * kBicgILP)
#define BICG_EACH(u) _Pragma("unroll") for (int u = 0; u < kBicgILP; ++u)
#define BICG_AT(base, u) min(base + (int64_t)(u) * kReduceThreads, n - 1)
#define BICG_ON(base, u) (base + (int64_t)(u) * kReduceThreads < n)

// r = b - Ax0 (ax = A x0), r^ = r; pairs (r^.r, r.r) and (b.b, 0)
template <typename V>
__global__ __launch_bounds__(kReduceThreads) void bicg_init_kernel(
    const V* __restrict__ b, const V* __restrict__ ax, V* __restrict__ r, V* __restrict__ rh,
    int64_t n, double* __restrict__ part_r, double* __restrict__ part_b) {
  double rr = 0.0, bb = 0.0;
  BICG_PASS(base) {
    V bv[kBicgILP], av[kBicgILP];
    BICG_EACH(u) {
      bv[u] = b[BICG_AT(base, u)];
      av[u] = ax[BICG_AT(base, u)];
    }
    BICG_EACH(u) if (BICG_ON(base, u)) {
      const V ri = bv[u] - av[u];
      r[BICG_AT(base, u)] = ri;
      rh[BICG_AT(base, u)] = ri;
      rr += (double)ri * (double)ri;
      bb += (double)bv[u] * (double)bv[u];
    }
  }
  double rr2 = rr, z = 0.0;
  write_pair(part_r, rr, rr2);
  write_pair(part_b, bb, z);
}

// p_new from p (another buffer: hot columns' values are formed from p again)
template <typename V>
__global__ __launch_bounds__(kReduceThreads) void bicg_update_p_kernel(
    const V* __restrict__ r, const V* __restrict__ p, V* __restrict__ p_new,
    const V* __restrict__ v, int64_t n, int first, const double* __restrict__ pa_cur,
    const double* __restrict__ pa_prev, const double* __restrict__ pb_prev,
    const double* __restrict__ pc_prev, int G, const int32_t* __restrict__ hot_cols,
    int32_t hot_n, V* __restrict__ x_hot) {
  const int64_t h0 = (int64_t)blockIdx.x * kReduceThreads + threadIdx.x;
  const int64_t hstride = (int64_t)gridDim.x * kReduceThreads;
  if (first) {
    BICG_PASS(base) {
      V rv[kBicgILP];
      BICG_EACH(u) rv[u] = r[BICG_AT(base, u)];
      BICG_EACH(u) if (BICG_ON(base, u)) p_new[BICG_AT(base, u)] = rv[u];
    }
    for (int64_t h = h0; h < hot_n; h += hstride) x_hot[h] = r[hot_cols[h]];
    return;
  }
  const double* const parts[4] = {pa_cur, pa_prev, pb_prev, pc_prev};
  double t[8];  // rho, rr; rho_prev, -; (r^, v), -; (t, s), (t, t)
  sum_pairs<4>(parts, G, t);
  const double rho = t[0], rho_prev = t[2];
  const double alpha_prev = safe_div(rho_prev, t[4]);
  const double omega_prev = safe_div(t[6], t[7]);
  const double beta = safe_div(rho, rho_prev) * safe_div(alpha_prev, omega_prev);
  const V bt = (V)beta, om = (V)omega_prev;
  BICG_PASS(base) {
    V rv[kBicgILP], pv[kBicgILP], vv[kBicgILP];
    BICG_EACH(u) {
      rv[u] = r[BICG_AT(base, u)];
      pv[u] = p[BICG_AT(base, u)];
      vv[u] = v[BICG_AT(base, u)];
    }
    BICG_EACH(u) if (BICG_ON(base, u))
      p_new[BICG_AT(base, u)] = rv[u] + bt * (pv[u] - om * vv[u]);
  }
  for (int64_t h = h0; h < hot_n; h += hstride) {
    const int64_t c = hot_cols[h];
    x_hot[h] = r[c] + bt * (p[c] - om * v[c]);
  }
}

// pairs (a.b, 0)
template <typename V>
__global__ __launch_bounds__(kReduceThreads) void bicg_dot1_kernel(
    const V* __restrict__ a, const V* __restrict__ b, int64_t n, double* __restrict__ part) {
  double d = 0.0, z = 0.0;
  BICG_PASS(base) {
    V av[kBicgILP], bv[kBicgILP];
    BICG_EACH(u) {
      av[u] = a[BICG_AT(base, u)];
      bv[u] = b[BICG_AT(base, u)];
    }
    BICG_EACH(u) if (BICG_ON(base, u)) d += (double)av[u] * (double)bv[u];
  }
  write_pair(part, d, z);
}

template <typename V>
__global__ __launch_bounds__(kReduceThreads) void bicg_update_s_kernel(
    const V* __restrict__ r, const V* __restrict__ v, V* __restrict__ s, int64_t n,
    const double* __restrict__ pa_cur, const double* __restrict__ pb_cur, int G,
    const int32_t* __restrict__ hot_cols, int32_t hot_n, V* __restrict__ x_hot) {
  const double* const parts[2] = {pa_cur, pb_cur};
  double t[4];  // rho, rr; (r^, v), -
  sum_pairs<2>(parts, G, t);
  const V al = (V)safe_div(t[0], t[2]);
  BICG_PASS(base) {
    V rv[kBicgILP], vv[kBicgILP];
    BICG_EACH(u) {
      rv[u] = r[BICG_AT(base, u)];
      vv[u] = v[BICG_AT(base, u)];
    }
    BICG_EACH(u) if (BICG_ON(base, u)) s[BICG_AT(base, u)] = rv[u] - al * vv[u];
  }
  for (int64_t h = (int64_t)blockIdx.x * kReduceThreads + threadIdx.x; h < hot_n;
       h += (int64_t)gridDim.x * kReduceThreads) {
    const int64_t c = hot_cols[h];
    x_hot[h] = r[c] - al * v[c];
  }
}

// pairs (t.s, t.t)
template <typename V>
__global__ __launch_bounds__(kReduceThreads) void bicg_dot2_kernel(
    const V* __restrict__ t, const V* __restrict__ s, int64_t n, double* __restrict__ part) {
  double ts = 0.0, tt = 0.0;
  BICG_PASS(base) {
    V tv[kBicgILP], sv[kBicgILP];
    BICG_EACH(u) {
      tv[u] = t[BICG_AT(base, u)];
      sv[u] = s[BICG_AT(base, u)];
    }
    BICG_EACH(u) if (BICG_ON(base, u)) {
      const double ti = (double)tv[u];
      ts += ti * (double)sv[u];
      tt += ti * ti;
    }
  }
  write_pair(part, ts, tt);
}

template <typename V>
__global__ __launch_bounds__(kReduceThreads) void bicg_update_xr_kernel(
    V* __restrict__ x, const V* __restrict__ p, const V* __restrict__ s, const V* __restrict__ t,
    V* __restrict__ r, const V* __restrict__ rh, int64_t n, const double* __restrict__ pa_cur,
    const double* __restrict__ pb_cur, const double* __restrict__ pc_cur, int G,
    double* __restrict__ pa_next) {
  const double* const parts[3] = {pa_cur, pb_cur, pc_cur};
  double q[6];  // rho, rr; (r^, v), -; (t, s), (t, t)
  sum_pairs<3>(parts, G, q);
  const V al = (V)safe_div(q[0], q[2]);
  const V om = (V)safe_div(q[4], q[5]);
  double rhr = 0.0, rr2 = 0.0;
  BICG_PASS(base) {
    V xv[kBicgILP], pv[kBicgILP], sv[kBicgILP], tv[kBicgILP], hv[kBicgILP];
    BICG_EACH(u) {
      xv[u] = x[BICG_AT(base, u)];
      pv[u] = p[BICG_AT(base, u)];
      sv[u] = s[BICG_AT(base, u)];
      tv[u] = t[BICG_AT(base, u)];
      hv[u] = rh[BICG_AT(base, u)];
    }
    BICG_EACH(u) if (BICG_ON(base, u)) {
      x[BICG_AT(base, u)] = xv[u] + al * pv[u] + om * sv[u];
      const V ri = sv[u] - om * tv[u];
      r[BICG_AT(base, u)] = ri;
      rhr += (double)hv[u] * (double)ri;
      rr2 += (double)ri * (double)ri;
    }
  }
  write_pair(pa_next, rhr, rr2);
}

#undef BICG_PASS
#undef BICG_EACH
#undef BICG_AT
#undef BICG_ON

int bicg_grid(int64_t n) { return pr_reduce_grid(n); }

template <typename V>
static hipError_t bicg_step_t(const BicgArgs& a, int stage, hipStream_t st) {
  const dim3 g((unsigned)a.G), b(kReduceThreads);
  const int64_t n = a.n;
  V* x = static_cast<V*>(a.x);
  V* r = static_cast<V*>(a.r);
  V* rh = static_cast<V*>(a.rh);
  V* p = static_cast<V*>(a.p);
  V* xh = static_cast<V*>(a.x_hot);
  V* v = static_cast<V*>(a.v);
  V* s = static_cast<V*>(a.s);
  V* t = static_cast<V*>(a.t);
  switch (stage) {
    case kBicgInit:
      hipLaunchKernelGGL(bicg_init_kernel<V>, g, b, 0, st, static_cast<const V*>(a.b), t, r, rh,
                         n, a.pa_next, a.pb_norm);
      break;
    case kBicgUpdateP:
      hipLaunchKernelGGL(bicg_update_p_kernel<V>, g, b, 0, st, r,
                         static_cast<const V*>(a.p_prev), p, v, n, a.first, a.pa_cur, a.pa_prev,
                         a.pb_prev, a.pc_prev, a.G, a.hot_cols, a.hot_n, xh);
      break;
    case kBicgDot1:
      hipLaunchKernelGGL(bicg_dot1_kernel<V>, g, b, 0, st, rh, v, n, a.pb_cur);
      break;
    case kBicgUpdateS:
      hipLaunchKernelGGL(bicg_update_s_kernel<V>, g, b, 0, st, r, v, s, n, a.pa_cur, a.pb_cur,
                         a.G, a.hot_cols, a.hot_n, xh);
      break;
    case kBicgDot2:
      hipLaunchKernelGGL(bicg_dot2_kernel<V>, g, b, 0, st, t, s, n, a.pc_cur);
      break;
    case kBicgUpdateXR:
      hipLaunchKernelGGL(bicg_update_xr_kernel<V>, g, b, 0, st, x, p, s, t, r, rh, n, a.pa_cur,
                         a.pb_cur, a.pc_cur, a.G, a.pa_next);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_bicg(int dtype, const BicgArgs& a, int stage, hipStream_t st) {
  return dtype == 0 ? bicg_step_t<float>(a, stage, st) : bicg_step_t<double>(a, stage, st);
}

}  // namespace merbit
