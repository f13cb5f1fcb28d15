// Pure-state steps of a closed model (Sec. IV.B: one photon on the plane of
// cavities without leakage).  With no decoherence operator acting on the
// basis the dissipator and the sink vanish and a pure start stays pure:
// rho_k = psi_k psi_k^dag, and the step's rotation U rho U^dag followed by
// the trace renormalisation is psi <- U psi / |psi| -- O(N^2) work per step
// instead of the two O(N^3) products.
//
// pure_step_kernel: one wavefront per row i of dU (= U - I, the context's
// propagator planes, ld x ld, zero padded) for each of NV vectors:
//   y_v[i] = (x_v[i] + sum_j dU[i][j] x_v[j]) / |x_v|.
// The row streams from HBM in 16-byte loads (coalesced: lane l of the wave
// takes columns (64 m + l) E .. + E - 1 of chunk m); x is re-read from the
// caches by every row.  Each lane accumulates its columns in the storage
// type; the wave then sums the lane partials in FP64 (butterfly) and forms
// y in FP64.  |x_v|^2 is summed in FP64 by every wave over the x elements it
// loads (all of x, in the same lane partition and order in every wave), so
// every row divides by the bitwise-same norm without any cross-workgroup
// step.  Rows and columns >= n are padding: x is read as zero there and the
// padding rows of y are written as zero.
//
// pure_series_kernel: where the context has the propagator's series
// (series_tile.hpp), all steps of a call in one launch, one workgroup per
// vector.  The vector and the terms stay on the compute unit: x, the sums and the
// first C entries of each row in registers, the series' v in LDS (real and
// imaginary part of a state side by side), so a step is `order` gather sweeps with
// one barrier each (v alternates between two buffers where both fit).  Rows of more
// than C entries (2 to 12, pure_shape) read the rest from memory in every term, and
// past N = 4096 the registers do not hold a lane's share (scratch per lane 84 bytes
// FP32 and 116 FP64 up to N = 5120, 290 and 370 past it; 12 to 28 from 3073 to
// 4096); elsewhere a step has no memory traffic, and the latency of that chain
// bounds it.  N = 4131 plane FP32 (seven terms): 23.3 us per step with dU streamed
// from HBM (136 MB per step at 5.9 TB/s), 6.4 so.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <string>
#include <utility>
#include <vector>

#include "ctx.hpp"
#include "device.hpp"
#include "lane_sums.hpp"
#include "lds_barrier.hpp"
#include "model.hpp"
#include "qme.h"

namespace qme {

static constexpr int kPureThreads = 128;   // two rows per workgroup
static constexpr int kPureLoads = 2;       // 16-byte loads per lane, row plane and pass

template <typename T>
struct alignas(16) Pack16 {
  T v[16 / sizeof(T)];
};

template <typename T>
__device__ __forceinline__ Pack16<T> load16(const T *p) {
  return *reinterpret_cast<const Pack16<T> *>(p);
}

template <typename T, int NV>
__global__ __launch_bounds__(kPureThreads) void pure_step_kernel(PureArgs<T> p) {
  constexpr int E = 16 / int(sizeof(T));
  constexpr int M = kPureLoads;
  constexpr int PASS = 64 * E * M;   // columns per pass of a wave: 512 FP32, 256 FP64
  const int lane = threadIdx.x & 63;
  const int64_t row = int64_t(blockIdx.x) * (kPureThreads / 64) + (threadIdx.x >> 6);
  if (row >= p.ld) return;
  if (row >= p.n) {
    if (lane < NV) {
      p.y_re[lane * p.ld + row] = T(0);
      p.y_im[lane * p.ld + row] = T(0);
    }
    return;
  }
  const T *ur = p.u_re + row * p.ld;
  const T *ui = p.u_im + row * p.ld;
  T acc_re[NV], acc_im[NV];
  double nrm[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    acc_re[v] = acc_im[v] = T(0);
    nrm[v] = 0.0;
  }
  for (int64_t c0 = 0; c0 < p.ld; c0 += PASS) {
    Pack16<T> a[M], b[M], xr[NV][M], xi[NV][M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int64_t col = c0 + int64_t(m * 64 + lane) * E;
      if (col < p.ld) {
        a[m] = load16(ur + col);
        b[m] = load16(ui + col);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          xr[v][m] = load16(p.x_re + v * p.ld + col);
          xi[v][m] = load16(p.x_im + v * p.ld + col);
        }
      } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          a[m].v[e] = b[m].v[e] = T(0);
#pragma unroll
          for (int v = 0; v < NV; ++v) xr[v][m].v[e] = xi[v][m].v[e] = T(0);
        }
      }
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int64_t col = c0 + int64_t(m * 64 + lane) * E;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const bool in = col + e < p.n;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const T x_re = in ? xr[v][m].v[e] : T(0);
          const T x_im = in ? xi[v][m].v[e] : T(0);
          nrm[v] += double(x_re) * double(x_re) + double(x_im) * double(x_im);
          acc_re[v] = fma(a[m].v[e], x_re, acc_re[v]);
          acc_re[v] = fma(-b[m].v[e], x_im, acc_re[v]);
          acc_im[v] = fma(a[m].v[e], x_im, acc_im[v]);
          acc_im[v] = fma(b[m].v[e], x_re, acc_im[v]);
        }
      }
    }
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    double sr = double(acc_re[v]), si = double(acc_im[v]), sn = nrm[v];
    for (int off = 32; off > 0; off >>= 1) {
      sr += __shfl_xor(sr, off);
      si += __shfl_xor(si, off);
      sn += __shfl_xor(sn, off);
    }
    if (lane == v) {
      const double scale = 1.0 / sqrt(sn);
      const int64_t o = v * p.ld + row;
      p.y_re[o] = T(scale * (double(p.x_re[o]) + sr));
      p.y_im[o] = T(scale * (double(p.x_im[o]) + si));
    }
  }
}

template <typename T>
struct PureSeriesArgs {
  T *re, *im;                // [vector][ld], updated in place
  int64_t ld;
  int32_t n, order, entry_bytes;
  const int32_t *slot_col, *slice_off, *entry_at;
  const T *entry_val;
  const double *phase;       // e^{i shift dt} - 1 per state
  int32_t varied;            // whether it differs between states
  double ratio[kSeriesMaxOrder + 1];
  int64_t steps;
};

// Waves of S slices of 64 states, the first C entries of each slice in
// registers (FP64 with many slices: the slots packed in pairs).  TWO: two
// buffers of v.
template <typename T, int S, int C, int NT, bool TWO>
__global__ __launch_bounds__(NT, NT / 256) void pure_series_kernel(PureSeriesArgs<T> p) {
  typedef T cplx __attribute__((ext_vector_type(2)));
  constexpr int U = int(sizeof(cplx));
  constexpr int W = NT / 64;
  constexpr int K = sizeof(T) == 8 && S >= 4 ? 2 : 1;   // slots per register
  extern __shared__ __align__(16) unsigned char lds[];
  const int tid = int(threadIdx.x), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = p.n, slices = (n + 63) >> 6;
  const int buffer = slices * 64 * U;
  double *s_norm = reinterpret_cast<double *>(lds + (TWO ? 2 : 1) * buffer);   // [2][4 W]
  T *re = p.re + int64_t(blockIdx.x) * p.ld, *im = p.im + int64_t(blockIdx.x) * p.ld;

  int off[S + 1];
#pragma unroll
  for (int s = 0; s <= S; ++s) off[s] = p.slice_off[min(wave * S + s, slices)];
  unsigned at[S][(C + K - 1) / K];
  T val[S][C];
  cplx x[S];
  int col[S];
  const int scale_at = p.entry_bytes;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int slot = (wave * S + s) * 64 + lane;
    col[s] = slot < n ? p.slot_col[slot] : -1;
    const int c = max(col[s], 0);
    x[s][0] = col[s] < 0 ? T(0) : re[c];
    x[s][1] = col[s] < 0 ? T(0) : im[c];
#pragma unroll
    for (int i = 0; i < (C + K - 1) / K; ++i) at[s][i] = 0;
#pragma unroll
    for (int i = 0; i < C; ++i) {
      // (an entry past the slice's last: slot 0, times zero)
      const bool in = off[s] + i < off[s + 1];
      const int64_t e = int64_t(in ? off[s] + i : 0) * 64 + lane;
      const unsigned slot_i = unsigned(in ? p.entry_at[e] / scale_at : 0);
      at[s][i / K] |= K == 1 ? slot_i * U : slot_i << (16 * (i % K));
      val[s][i] = in ? p.entry_val[e] : T(0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  auto slot_at = [&](int s, int i) {
    const unsigned a = at[s][i / K];
    return int(K == 1 ? a : (i % K ? a >> 16 : a & 65535u) * U);
  };
  auto store = [&](int s, int to, const cplx &u) {
    const int slice = wave * S + s;
    if (slice < slices)
      *reinterpret_cast<cplx *>(lds + to + (slice * 64 + lane) * U) = u;
  };
  const double q0_re = p.phase[0], q0_im = -p.phase[1], w1 = p.ratio[1];

  int flip = 0;
  for (int64_t step = 0; step < p.steps; ++step) {
    double *norms = s_norm + int(step & 1) * 4 * W;   // per wave, one of each row of lanes
    double norm = 0.0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      store(s, TWO ? flip * buffer : 0, x[s]);
      norm += double(x[s][0]) * double(x[s][0]) + double(x[s][1]) * double(x[s][1]);
    }
    cplx t[S];
    for (int k = p.order; k >= 1; --k) {
      lds_barrier();
      const unsigned char *v = lds + (TWO ? flip * buffer : 0);
      if constexpr (K == 2) {
        // (the packed slots are unpacked here, in each term: as invariants of
        // the loop they would take twice the registers)
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
          for (int i = 0; i < (C + K - 1) / K; ++i) asm volatile("" : "+v"(at[s][i]));
      }
#pragma unroll
      for (int s = 0; s < S; ++s) {
        t[s] = cplx(T(0));
        // (four entries' gathers in flight at a time)
#pragma unroll
        for (int i0 = 0; i0 < C; i0 += 4) {
          if (i0 > 0 && off[s] + i0 >= off[s + 1]) break;
          cplx g[4];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (i0 + i < C) g[i] = *reinterpret_cast<const cplx *>(v + slot_at(s, i0 + i));
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (i0 + i < C) {
              t[s][0] = fma(val[s][i0 + i], g[i][0], t[s][0]);
              t[s][1] = fma(val[s][i0 + i], g[i][1], t[s][1]);
            }
        }
        for (int e = off[s] + C; e < off[s + 1]; ++e) {
          const int64_t o = int64_t(e) * 64 + lane;
          const cplx h = *reinterpret_cast<const cplx *>(v + p.entry_at[o] / scale_at * U);
          const T w = p.entry_val[o];
          t[s][0] = fma(w, h[0], t[s][0]);
          t[s][1] = fma(w, h[1], t[s][1]);
        }
      }
      if (k == p.order) {
        // |x|^2, while the other waves gather (read behind a later barrier)
        norm = row_sum(norm);
        if ((lane & 15) == 0) norms[wave * 4 + (lane >> 4)] = norm;
      }
      flip ^= 1;
      if (k == 1) break;
      if constexpr (!TWO) lds_barrier();
      const T w = T(p.ratio[k]);   // v <- x - i w K v
#pragma unroll
      for (int s = 0; s < S; ++s) {
        cplx u;
        u[0] = fma(w, t[s][1], x[s][0]);
        u[1] = fma(-w, t[s][0], x[s][1]);
        store(s, TWO ? flip * buffer : 0, u);
      }
    }
    // (one buffer: every wave has read v before the next step writes it; one
    // term: the norms have had no barrier yet)
    if (!TWO || p.order == 1) lds_barrier();
    static_assert(W == 4 || W == 16, "a row of lanes, or four, sums the norms");
    double sum = row_sum(norms[lane & (4 * W - 1)]);
    if constexpr (W == 16) {
      sum += __shfl_xor(sum, 16);
      sum += __shfl_xor(sum, 32);
    }
    const double scale = 1.0 / sqrt(sum);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      double q_re = q0_re, q_im = q0_im;
      if (p.varied) {
        q_re = p.phase[2 * max(col[s], 0)];
        q_im = -p.phase[2 * max(col[s], 0) + 1];
      }
      const double dr = w1 * double(t[s][1]), di = -w1 * double(t[s][0]);
      const double yr = double(x[s][0]) + dr, yi = double(x[s][1]) + di;
      x[s][0] = T(scale * (double(x[s][0]) + (dr + (q_re * yr - q_im * yi))));
      x[s][1] = T(scale * (double(x[s][1]) + (di + (q_re * yi + q_im * yr))));
      // (one state's FP64 values live at a time)
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (col[s] >= 0) {
      re[col[s]] = x[s][0];
      im[col[s]] = x[s][1];
    }
}

constexpr int64_t kPureStepsPerLaunch = 2048;

template <typename T, int S, int C, int NT, bool TWO>
static hipError_t launch_series_buffers(const PureSeriesArgs<T> &a, int nv, size_t lds, hipStream_t s) {
  const auto kernel = pure_series_kernel<T, S, C, NT, TWO>;
  if (lds > 48 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
  }
  for (int64_t done = 0; done < a.steps; done += kPureStepsPerLaunch) {
    PureSeriesArgs<T> b = a;
    b.steps = std::min(kPureStepsPerLaunch, a.steps - done);
    hipLaunchKernelGGL(kernel, dim3(unsigned(nv)), dim3(NT), lds, s, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T, int S, int C, int NT>
static hipError_t launch_series_shape(const PureSeriesArgs<T> &a, int nv, hipStream_t s) {
  const size_t buffer = size_t(a.n + 63) / 64 * 64 * 2 * sizeof(T), norm = 8 * (NT / 64) * sizeof(double);
  if (2 * buffer + norm <= 163840)
    return launch_series_buffers<T, S, C, NT, true>(a, nv, 2 * buffer + norm, s);
  return launch_series_buffers<T, S, C, NT, false>(a, nv, buffer + norm, s);
}

// The registers that a lane can give its rows' entries (128 at four waves per
// SIMD) set C: rows with more entries read the rest from memory in each term.
struct PureShape {
  int slices, kept, threads;   // S, C, NT
};
static constexpr PureShape pure_shape(int64_t n, bool fp32) {
  if (n <= 256) return {1, fp32 ? 12 : 8, 256};
  if (n <= 1024) return {1, fp32 ? 12 : 8, 1024};
  if (n <= 2048) return {2, fp32 ? 12 : 6, 1024};
  if (n <= 3072) return {3, fp32 ? 8 : 4, 1024};
  if (n <= 4096) return {4, fp32 ? 6 : 4, 1024};
  if (n <= 5120) return {5, fp32 ? 4 : 3, 1024};
  return {8, 2, 1024};
}

// A step is a chain of `order` terms on one compute unit, each as long as the
// wave with the most entries past those in registers: they are read one after
// another, 0.18 us each from the L2, 0.38 where they no longer fit it (4 MB).  The
// dense step streams dU through the whole device, or is one launch.  Fits to steps
// timed with rows of 2 to 400 entries and a star at N = 40 ... 4097; series /
// dense, us per step: rows of 2 at N = 513 FP32 2.8 / 3.9, of 8 at 2048 5.4 / 5.5
// (scattered 8.9 / 5.6), of 32 at 2048 64 / 5.5 and 4096 169 / 21.6, of 200 at 4096
// 2726 / 21.6; star N = 65 50 / 3.6, 2048 2564 / 5.8; FP64 rows of 4 at 4096 14.5 /
// 39.9, of 8 at 1025 12.7 / 5.4.
double pure_series_us(const SeriesPlan &p, int64_t n, int elem) {
  const PureShape f = pure_shape(n, elem == 4);
  const int64_t slices = int64_t(p.slice_off.size()) - 1;
  int64_t longest = 0, more = 0, kept = 0;
  for (int64_t q0 = 0; q0 < slices; q0 += f.slices) {
    int64_t wave = 0;
    for (int64_t q = q0; q < std::min(slices, q0 + f.slices); ++q) {
      const int64_t len = p.slice_off[size_t(q) + 1] - p.slice_off[size_t(q)];
      wave += std::max<int64_t>(0, len - f.kept);
      kept += std::min<int64_t>(len, f.kept);
    }
    more += wave;
    longest = std::max(longest, wave);
  }
  const bool in_l2 = more * 64 * (4 + elem) <= 4 << 20;
  const double lds = double(kept) * 64.0 * 2.0 * elem / (128.0 * 2400.0) * (0.55 + 0.95 * p.scattered);
  const double latency = f.threads == 256 ? 0.23 : 0.2 + 0.1 * f.slices + (elem == 8 && f.slices >= 4 ? 0.2 : 0.0);
  return p.order * (latency + lds + (in_l2 ? 0.18 : 0.38) * double(longest));
}

// Measured (MI355X, us per step in calls of 20).
double pure_dense_us(int64_t n, int elem) {
  static constexpr double kN[6] = {64, 256, 512, 1024, 2048, 4096};
  static constexpr double kFp32[6] = {3.1, 3.3, 3.7, 4.5, 5.6, 21.5};
  static constexpr double kFp64[6] = {3.0, 3.4, 3.9, 5.1, 11.7, 40.0};
  return interpolate_us(kN, elem == 4 ? kFp32 : kFp64, 6, 2.0, double(n));
}

template <typename T>
static hipError_t launch_pure_series(const PureSeriesArgs<T> &a, int nv, hipStream_t s) {
  constexpr bool F = sizeof(T) == 4;
  if (a.n < 1 || a.n > kSeriesMaxN || a.order < 1 || a.order > kSeriesMaxOrder || nv < 1)
    return hipErrorInvalidValue;
  // the shape that pure_shape gives for the largest N of each line
  auto run = [&](auto top) {
    constexpr PureShape f = pure_shape(decltype(top)::value, F);
    return launch_series_shape<T, f.slices, f.kept, f.threads>(a, nv, s);
  };
  if (a.n <= 256) return run(std::integral_constant<int64_t, 256>{});
  if (a.n <= 1024) return run(std::integral_constant<int64_t, 1024>{});
  if (a.n <= 2048) return run(std::integral_constant<int64_t, 2048>{});
  if (a.n <= 3072) return run(std::integral_constant<int64_t, 3072>{});
  if (a.n <= 4096) return run(std::integral_constant<int64_t, 4096>{});
  if (a.n <= 5120) return run(std::integral_constant<int64_t, 5120>{});
  return run(std::integral_constant<int64_t, kSeriesMaxN>{});
}

template <typename T, int NV>
static hipError_t launch_nv(const PureArgs<T> &a, hipStream_t s) {
  const unsigned blocks = unsigned(a.ld / (kPureThreads / 64));
  hipLaunchKernelGGL((pure_step_kernel<T, NV>), dim3(blocks), dim3(kPureThreads), 0, s, a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_pure_step(const PureArgs<T> &a, int nv, hipStream_t s) {
  if (a.n < 1 || a.ld < a.n || a.ld % (kPureThreads / 64) != 0 || a.ld % (16 / sizeof(T)) != 0)
    return hipErrorInvalidValue;
  switch (nv) {
    case 1: return launch_nv<T, 1>(a, s);
    case 2: return launch_nv<T, 2>(a, s);
    case 3: return launch_nv<T, 3>(a, s);
    case 4: return launch_nv<T, 4>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template hipError_t launch_pure_step<float>(const PureArgs<float> &, int, hipStream_t);
template hipError_t launch_pure_step<double>(const PureArgs<double> &, int, hipStream_t);

}  // namespace qme

using namespace qme;

#define PURE_OK(call)                                                         \
  do {                                                                        \
    hipError_t e_ = (call);                                                   \
    if (e_ != hipSuccess) {                                                   \
      set_error(std::string(#call) + ": " + hipGetErrorString(e_));           \
      return QME_E_DEVICE;                                                    \
    }                                                                         \
  } while (0)

namespace {

size_t pure_bytes(const qme_ctx *c, int32_t n_vec) {
  const size_t b = 2 * size_t(n_vec) * size_t(c->ld) * size_t(c->elem);
  return (b + 255) / 256 * 256;
}

// Validation shared by the pure-state calls: context, vector count and
// precision (FP32 / FP64 storage; BF16X3 contexts have no pure form).
qme_status pure_check(const qme_ctx *c, int32_t n_vec) {
  if (!c) { set_error("ctx is NULL"); return QME_E_ARG; }
  if (n_vec < 1 || n_vec > QME_PURE_MAX_VECTORS) {
    set_error("n_vec must be in [1, QME_PURE_MAX_VECTORS]");
    return QME_E_ARG;
  }
  if (c->precision == QME_BF16X3) {
    set_error("pure-state steps run in FP32 or FP64 contexts");
    return QME_E_UNSUPPORTED;
  }
  return QME_OK;
}

// No decoherence operator acts on the basis: no gather channel, and every
// rate-weighted A^dag A diagonal and leak weight is zero.
bool closed_model(const qme_ctx *c) {
  if (c->jt.n_gather != 0) return false;
  for (double x : c->jt.d)
    if (x != 0.0) return false;
  for (double x : c->jt.leak)
    if (x != 0.0) return false;
  return true;
}

template <typename T>
qme_status pure_run(qme_ctx *c, void *state, int32_t n_vec, int64_t n_steps, void *ws,
                    hipStream_t s) {
  const size_t plane = size_t(n_vec) * size_t(c->ld);
  T *a = static_cast<T *>(state), *b = static_cast<T *>(ws);
  if (c->series_order > 0 && (c->products == 1 || (c->products < 0 && c->pure_series_faster))) {
    PureSeriesArgs<T> p{a, a + plane, c->ld, int32_t(c->n), c->series_order,
                        series_slot_bytes(c->n), c->s_col, c->s_off, c->s_at,
                        static_cast<const T *>(c->s_val), c->s_phase, c->series_phase ? 1 : 0, {}, n_steps};
    for (int k = 1; k <= c->series_order; ++k) p.ratio[k] = c->series_ratio[k];
    PURE_OK(launch_pure_series<T>(p, n_vec, s));
    return QME_OK;
  }
  if (n_steps % 2) {
    // odd count: start from a copy in the workspace so the last step writes the state
    PURE_OK(hipMemcpyAsync(ws, state, 2 * plane * sizeof(T), hipMemcpyDeviceToDevice, s));
    std::swap(a, b);
  }
  for (int64_t k = 0; k < n_steps; ++k) {
    PureArgs<T> args{a, a + plane, b, b + plane, static_cast<const T *>(c->du_re),
                     static_cast<const T *>(c->du_im), c->ld, c->n};
    PURE_OK(launch_pure_step<T>(args, n_vec, s));
    std::swap(a, b);
  }
  return QME_OK;
}

}  // namespace

extern "C" qme_status qme_pure_layout(const qme_ctx *c, int32_t n_vec, size_t *state_bytes,
                                      size_t *workspace_bytes) {
  set_error("");
  const qme_status st = pure_check(c, n_vec);
  if (st != QME_OK) return st;
  if (state_bytes) *state_bytes = pure_bytes(c, n_vec);
  if (workspace_bytes) *workspace_bytes = pure_bytes(c, n_vec);
  return QME_OK;
}

extern "C" qme_status qme_pure_set(const qme_ctx *c, void *state, int32_t n_vec,
                                   const double *psi_re, const double *psi_im, void *hip_stream) {
  try {
    set_error("");
    qme_status st = pure_check(c, n_vec);
    if (st != QME_OK) return st;
    if (!state || !psi_re || !psi_im) { set_error("NULL argument"); return QME_E_ARG; }
    st = check_device(c);
    if (st != QME_OK) return st;
    const size_t plane = size_t(n_vec) * size_t(c->ld);
    std::vector<char> buf(pure_bytes(c, n_vec), 0);
    for (int32_t v = 0; v < n_vec; ++v) {
      double norm = 0.0;
      for (int64_t i = 0; i < c->n; ++i) {
        const double xr = psi_re[size_t(v) * c->n + i], xi = psi_im[size_t(v) * c->n + i];
        if (!std::isfinite(xr) || !std::isfinite(xi)) { set_error("psi is not finite"); return QME_E_ARG; }
        norm += xr * xr + xi * xi;
        const size_t o = size_t(v) * c->ld + i;
        if (c->elem == 8) {
          reinterpret_cast<double *>(buf.data())[o] = xr;
          reinterpret_cast<double *>(buf.data())[plane + o] = xi;
        } else {
          reinterpret_cast<float *>(buf.data())[o] = float(xr);
          reinterpret_cast<float *>(buf.data())[plane + o] = float(xi);
        }
      }
      if (!(norm > 0.0)) { set_error("psi has a zero vector"); return QME_E_ARG; }
    }
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    PURE_OK(hipMemcpyAsync(state, buf.data(), buf.size(), hipMemcpyHostToDevice, s));
    PURE_OK(hipStreamSynchronize(s));
    return QME_OK;
  } catch (const std::bad_alloc &) {
    set_error("out of host memory");
    return QME_E_SIZE;
  } catch (const std::exception &e) {
    set_error(std::string("internal error: ") + e.what());
    return QME_E_STATE;
  }
}

extern "C" qme_status qme_pure_get(const qme_ctx *c, const void *state, int32_t n_vec,
                                   double *psi_re, double *psi_im, void *hip_stream) {
  try {
    set_error("");
    qme_status st = pure_check(c, n_vec);
    if (st != QME_OK) return st;
    if (!state) { set_error("NULL argument"); return QME_E_ARG; }
    st = check_device(c);
    if (st != QME_OK) return st;
    const size_t plane = size_t(n_vec) * size_t(c->ld);
    std::vector<char> buf(pure_bytes(c, n_vec));
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    PURE_OK(hipMemcpyAsync(buf.data(), state, buf.size(), hipMemcpyDeviceToHost, s));
    PURE_OK(hipStreamSynchronize(s));
    for (int32_t v = 0; v < n_vec; ++v)
      for (int64_t i = 0; i < c->n; ++i) {
        const size_t o = size_t(v) * c->ld + i, dst = size_t(v) * c->n + i;
        const double xr = c->elem == 8 ? reinterpret_cast<double *>(buf.data())[o]
                                       : double(reinterpret_cast<float *>(buf.data())[o]);
        const double xi = c->elem == 8 ? reinterpret_cast<double *>(buf.data())[plane + o]
                                       : double(reinterpret_cast<float *>(buf.data())[plane + o]);
        if (psi_re) psi_re[dst] = xr;
        if (psi_im) psi_im[dst] = xi;
      }
    return QME_OK;
  } catch (const std::bad_alloc &) {
    set_error("out of host memory");
    return QME_E_SIZE;
  } catch (const std::exception &e) {
    set_error(std::string("internal error: ") + e.what());
    return QME_E_STATE;
  }
}

extern "C" qme_status qme_pure_step(qme_ctx *c, void *state, int32_t n_vec, int64_t n_steps,
                                    void *ws, void *hip_stream) {
  try {
    TraceRange range("qme_pure_step");
    set_error("");
    qme_status st = pure_check(c, n_vec);
    if (st != QME_OK) return st;
    if (!state || !ws) { set_error("NULL argument"); return QME_E_ARG; }
    if (n_steps < 0) { set_error("n_steps < 0"); return QME_E_ARG; }
    if ((reinterpret_cast<uintptr_t>(state) | reinterpret_cast<uintptr_t>(ws)) & 255) {
      set_error("state and workspace must be 256-byte aligned");
      return QME_E_ARG;
    }
    if (!closed_model(c)) {
      set_error("pure-state steps need a closed model (no decoherence operator acting on the basis)");
      return QME_E_STATE;
    }
    st = check_device(c);
    if (st != QME_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    return c->elem == 8 ? pure_run<double>(c, state, n_vec, n_steps, ws, s)
                        : pure_run<float>(c, state, n_vec, n_steps, ws, s);
  } catch (const std::bad_alloc &) {
    set_error("out of host memory");
    return QME_E_SIZE;
  } catch (const std::exception &e) {
    set_error(std::string("internal error: ") + e.what());
    return QME_E_STATE;
  }
}
