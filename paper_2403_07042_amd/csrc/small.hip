// Whole time steps of a small system (n <= 32) in one launch of one
// workgroup: the propagator increment and the state stay in LDS for every
// step, so a step costs no kernel launches and no HBM traffic.
//
// The step is the same as the tiled path's (Sec. II, Eqs. 2-3, with the
// "unitary evolution" products of Sec. IV.B):
//   T   = rho + dU rho                (rho Hermitian: B[k][j] = conj(rho[j][k]))
//   Z   = T + T conj(dU)              on and below the diagonal
//   trace / sink / renormalisation    FP64, the same reduction tree
//   rho' = scale * Herm(Z + dt D(Z))  FP64, written in both triangles
// Products accumulate in the storage type with scalar FMAs (k ascending);
// the decoherence arithmetic is operation-for-operation that of the tiled
// decoherence pass, so only the products' rounding order differs from it.
//
// small_rows_kernel: where the rows of dU have few entries (up to eight: states
// that H does not connect have none) and the channels are few.  One element per
// thread; a thread keeps what it needs of dU's rows, the decoherence factors
// and the gathers in registers for all steps, and every wave forms the trace
// itself, so a step is three LDS round trips with a barrier each (none for n <=
// 8: one wave).  What bounds it is the latency of that chain.  The general
// kernel reads dU and the tables from LDS again in every step and divides
// every element index by n: N = 8 Jaynes-Cummings 2.15 -> 0.44 us per step, N =
// 32 (FP32, three channels) 20.4 -> 1.6.
#include "device.hpp"
#include "lane_sums.hpp"
#include "lds_barrier.hpp"

#include <algorithm>

namespace qme {

constexpr int kSmallLd = kSmallN + 1;     // padded LDS row
constexpr int kSmallThreads = 256;
constexpr int kSmallGather = 16;          // channels whose tables are staged in LDS
constexpr int64_t kSmallStepsPerLaunch = 4096;

template <typename T>
__global__ __launch_bounds__(kSmallThreads) void small_steps_kernel(SmallArgs<T> p) {
  __shared__ T sU[2][kSmallN * kSmallLd];
  __shared__ T sA[2][kSmallN * kSmallLd];
  __shared__ T sB[2][kSmallN * kSmallLd];
  __shared__ double s_d[kSmallN], s_leak[kSmallN], s_trw[kSmallN];
  __shared__ int32_t s_pi[kSmallGather][kSmallN];
  __shared__ double s_cg[kSmallGather][kSmallN];
  __shared__ double s_scale;

  const int n = p.n, tid = threadIdx.x, nn = n * n;
  const int64_t ld = p.ld;
  const bool staged = p.n_gather <= kSmallGather;
  for (int e = tid; e < nn; e += kSmallThreads) {
    const int i = e / n, j = e - (e / n) * n;
    sU[0][i * kSmallLd + j] = p.u_re[i * ld + j];
    sU[1][i * kSmallLd + j] = p.u_im[i * ld + j];
    sA[0][i * kSmallLd + j] = p.re[i * ld + j];
    sA[1][i * kSmallLd + j] = p.im[i * ld + j];
  }
  for (int u = tid; u < n; u += kSmallThreads) {
    s_d[u] = p.d[u];
    s_leak[u] = p.leak[u];
    s_trw[u] = p.trw[u];
  }
  if (staged)
    for (int e = tid; e < p.n_gather * n; e += kSmallThreads) {
      const int j = e / n, u = e - (e / n) * n;
      s_pi[j][u] = p.pi[int64_t(j) * n + u];
      s_cg[j][u] = p.cg[int64_t(j) * n + u];
    }
  double sink = p.aux[0], rot = p.aux[1], lost = p.aux[2], steps = p.aux[3], scale = p.aux[4];
  __syncthreads();

  T(*rho)[kSmallN * kSmallLd] = sA;
  T(*tb)[kSmallN * kSmallLd] = sB;
  const double dt = p.dt;
  for (int64_t s = 0; s < p.steps; ++s) {
    // T = rho + dU rho
    for (int e = tid; e < nn; e += kSmallThreads) {
      const int i = e / n, j = e - (e / n) * n;
      T cr = T(0), ci = T(0);
      for (int k = 0; k < n; ++k) {
        const T ar = sU[0][i * kSmallLd + k], ai = sU[1][i * kSmallLd + k];
        const T mr = rho[0][j * kSmallLd + k], mi = rho[1][j * kSmallLd + k];
        cr = fma(ar, mr, cr);
        cr = fma(ai, mi, cr);
        ci = fma(ai, mr, ci);
        ci = fma(-ar, mi, ci);
      }
      tb[0][i * kSmallLd + j] = cr + rho[0][i * kSmallLd + j];
      tb[1][i * kSmallLd + j] = ci + rho[1][i * kSmallLd + j];
    }
    __syncthreads();
    // Z = T + T conj(dU), lower triangle, into rho's buffer (rho is dead)
    T(*z)[kSmallN * kSmallLd] = rho;
    for (int e = tid; e < nn; e += kSmallThreads) {
      const int i = e / n, j = e - (e / n) * n;
      if (j > i) continue;
      T cr = T(0), ci = T(0);
      for (int k = 0; k < n; ++k) {
        const T ar = tb[0][i * kSmallLd + k], ai = tb[1][i * kSmallLd + k];
        const T mr = sU[0][j * kSmallLd + k], mi = sU[1][j * kSmallLd + k];
        cr = fma(ar, mr, cr);
        cr = fma(ai, mi, cr);
        ci = fma(ai, mr, ci);
        ci = fma(-ar, mi, ci);
      }
      z[0][i * kSmallLd + j] = cr + tb[0][i * kSmallLd + j];
      z[1][i * kSmallLd + j] = ci + tb[1][i * kSmallLd + j];
    }
    __syncthreads();
    // trace, lost probability and renormalisation (wave 0; lanes >= n add 0)
    if (tid < 64) {
      double tr = 0.0, lo = 0.0, ro = 0.0;
      if (tid < n) {
        const int u = tid;
        const double zu = double(z[0][u * kSmallLd + u]);
        tr = s_trw[u] * zu;
        lo = s_leak[u] * zu;
        ro = zu;
      }
      for (int w = kSmallN / 2; w > 0; w >>= 1) {
        tr += __shfl_down(tr, w);
        lo += __shfl_down(lo, w);
        ro += __shfl_down(ro, w);
      }
      if (tid == 0) {
        sink = sink + dt * lo;
        steps = steps + 1.0;
        rot = ro;
        lost = lo;
        scale = (1.0 - sink) / tr;
        s_scale = scale;
      }
    }
    __syncthreads();
    // rho' = scale * (Z + dt D(Z)) on and below the diagonal, mirrored, into tb
    const double sc = s_scale;
    for (int e = tid; e < nn; e += kSmallThreads) {
      const int u = e / n, v = e - (e / n) * n;
      if (v > u) continue;
      const double zr = double(z[0][u * kSmallLd + v]), zi = double(z[1][u * kSmallLd + v]);
      const double f = 1.0 - 0.5 * dt * (s_d[u] + s_d[v]);
      double xr = f * zr, xi = f * zi;
      for (int j = 0; j < p.n_gather; ++j) {
        const int32_t pu = staged ? s_pi[j][u] : p.pi[int64_t(j) * n + u];
        const int32_t pv = staged ? s_pi[j][v] : p.pi[int64_t(j) * n + v];
        if (pu >= 0 && pv >= 0) {
          const double cu = staged ? s_cg[j][u] : p.cg[int64_t(j) * n + u];
          const double cv = staged ? s_cg[j][v] : p.cg[int64_t(j) * n + v];
          const double w = dt * cu * cv;
          double gr, gi;
          if (pu >= pv) {
            gr = double(z[0][pu * kSmallLd + pv]);
            gi = double(z[1][pu * kSmallLd + pv]);
          } else {
            gr = double(z[0][pv * kSmallLd + pu]);
            gi = -double(z[1][pv * kSmallLd + pu]);
          }
          xr += w * gr;
          xi += w * gi;
        }
      }
      xr *= sc;
      xi *= sc;
      if (u == v) xi = 0.0;
      tb[0][u * kSmallLd + v] = T(xr);
      tb[1][u * kSmallLd + v] = T(xi);
      if (u != v) {
        tb[0][v * kSmallLd + u] = T(xr);
        tb[1][v * kSmallLd + u] = T(-xi);
      }
    }
    __syncthreads();
    T(*t)[kSmallN * kSmallLd] = rho;
    rho = tb;
    tb = t;
  }
  for (int e = tid; e < nn; e += kSmallThreads) {
    const int i = e / n, j = e - (e / n) * n;
    p.re[i * ld + j] = rho[0][i * kSmallLd + j];
    p.im[i * ld + j] = rho[1][i * kSmallLd + j];
  }
  if (tid == 0) {
    p.aux[0] = sink;
    p.aux[1] = rot;
    p.aux[2] = lost;
    p.aux[3] = steps;
    p.aux[4] = scale;
  }
}

template <typename T>
__device__ __forceinline__ T __attribute__((ext_vector_type(2))) small_pair(T re, T im) {
  T v __attribute__((ext_vector_type(2)));
  v[0] = re;
  v[1] = im;
  return v;
}

// What one element's thread keeps for its decoherence step and the trace.
template <typename T, int G>
struct SmallElement {
  typedef T cplx __attribute__((ext_vector_type(2)));
  double f, gw[G];            // decay factor; per channel its weight (0: none)
  int ga[G];                  // and where its element lies, below the diagonal
  unsigned flip = 0;          // bit g: that element is the conjugate's
  int dw;
  double trw, leak, one;      // of the state whose diagonal this lane adds to the trace

  __device__ __forceinline__ void load(const SmallArgs<T> &p, int i, int j, int lane) {
    const int n = p.n;
    f = 1.0 - 0.5 * p.dt * (p.d[i] + p.d[j]);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      ga[g] = 0;
      gw[g] = 0.0;
      if (g < p.n_gather) {
        const int pu = p.pi[int64_t(g) * n + i], pv = p.pi[int64_t(g) * n + j];
        if (pu >= 0 && pv >= 0) {
          ga[g] = pu >= pv ? pu * kSmallLd + pv : pv * kSmallLd + pu;
          flip |= pu >= pv ? 0u : 1u << g;
          gw[g] = p.dt * p.cg[int64_t(g) * n + i] * p.cg[int64_t(g) * n + j];
        }
      }
    }
    const int w = n <= 16 ? lane & 15 : lane & 31;
    dw = w < n ? w * (kSmallLd + 1) : 0;
    trw = w < n ? p.trw[w] : 0.0;
    leak = w < n ? p.leak[w] : 0.0;
    one = w < n ? 1.0 : 0.0;
  }
  // Z + dt D(Z) of this element, z its own value, s_z the lower triangle
  __device__ __forceinline__ void decohere(const cplx &z, const cplx *s_z, double &xr, double &xi) const {
    xr = f * double(z[0]);
    xi = f * double(z[1]);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const cplx h = s_z[ga[g]];
      xr += gw[g] * double(h[0]);
      xi += gw[g] * ((flip >> g) & 1u ? -double(h[1]) : double(h[1]));
    }
  }
};

// The step's scalars, the same in every thread.
struct SmallScalars {
  double sink, rot, lost, steps, scale;
  template <typename T, int G>
  __device__ __forceinline__ void advance(const SmallArgs<T> &p, const SmallElement<T, G> &e,
                                          double zd) {
    auto total = [&](double x) {
      x = row_sum(x);
      return p.n <= 16 ? x : x + __shfl_xor(x, 16);
    };
    const double tr = total(e.trw * zd);
    lost = total(e.leak * zd);
    rot = total(e.one * zd);
    sink = sink + p.dt * lost;
    steps = steps + 1.0;
    scale = (1.0 - sink) / tr;
  }
};

// L: entries of a row of dU, G: gather channels, NT: threads (n * n at most).
template <typename T, int L, int G, int NT>
__global__ __launch_bounds__(NT) void small_rows_kernel(SmallArgs<T> p) {
  typedef T cplx __attribute__((ext_vector_type(2)));
  __shared__ cplx s_rho[kSmallN * kSmallLd], s_t[kSmallN * kSmallLd], s_z[kSmallN * kSmallLd];
  __shared__ int32_t s_k[kSmallN][L];
  __shared__ cplx s_u[kSmallN][L];
  const int n = p.n, tid = int(threadIdx.x), lane = tid & 63;
  const double dt = p.dt;
  // rows of dU without their zeros, in increasing k
  if (tid < n) {
    int c = 0;
    for (int k = 0; k < n; ++k) {
      const T ur = p.u_re[tid * p.ld + k], ui = p.u_im[tid * p.ld + k];
      if ((ur != T(0) || ui != T(0)) && c < L) {
        s_k[tid][c] = k;
        s_u[tid][c++] = small_pair<T>(ur, ui);
      }
    }
    for (; c < L; ++c) {
      s_k[tid][c] = 0;
      s_u[tid][c] = small_pair<T>(0, 0);
    }
  }
  const int i = tid / n, j = tid - i * n;
  const bool in = i < n, low = in && j <= i;
  const int e = in ? i * kSmallLd + j : 0, ei = in ? i : 0, ej = in ? j : 0;
  if (in) s_rho[e] = small_pair<T>(p.re[i * p.ld + j], p.im[i * p.ld + j]);
  lds_barrier();
  // this element's row i of dU against row j of rho, row i of T against row j
  // of dU
  int at1[L], at2[L];
  cplx u1[L], u2[L];
#pragma unroll
  for (int l = 0; l < L; ++l) {
    at1[l] = ej * kSmallLd + s_k[ei][l];
    u1[l] = s_u[ei][l];
    at2[l] = ei * kSmallLd + s_k[ej][l];
    u2[l] = s_u[ej][l];
  }
  SmallElement<T, G> el;
  el.load(p, ei, ej, lane);
  SmallScalars sc{p.aux[0], p.aux[1], p.aux[2], p.aux[3], p.aux[4]};

  cplx own = s_rho[e];
  for (int64_t s = 0; s < p.steps; ++s) {
    // T = rho + dU rho (rho Hermitian)
    T cr = T(0), ci = T(0);
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const cplx m = s_rho[at1[l]];
      cr = fma(u1[l][0], m[0], cr);
      cr = fma(u1[l][1], m[1], cr);
      ci = fma(u1[l][1], m[0], ci);
      ci = fma(-u1[l][0], m[1], ci);
    }
    const cplx t = small_pair<T>(cr + own[0], ci + own[1]);
    if (in) s_t[e] = t;
    lds_barrier();
    // Z = T + T conj(dU), lower triangle
    cr = ci = T(0);
#pragma unroll
    for (int l = 0; l < L; ++l) {
      const cplx a = s_t[at2[l]];
      cr = fma(a[0], u2[l][0], cr);
      cr = fma(a[1], u2[l][1], cr);
      ci = fma(a[1], u2[l][0], ci);
      ci = fma(-a[0], u2[l][1], ci);
    }
    const cplx z = small_pair<T>(cr + t[0], ci + t[1]);
    if (low) s_z[e] = z;
    lds_barrier();
    // trace, lost probability and renormalisation, in every wave
    const double zd = double(s_z[el.dw][0]);
    double xr, xi;
    el.decohere(z, s_z, xr, xi);
    sc.advance(p, el, zd);
    // rho' = scale * (Z + dt D(Z)) on and below the diagonal, mirrored
    if (low) {
      const T a = T(xr * sc.scale), b = i == j ? T(0) : T(xi * sc.scale);
      s_rho[e] = small_pair<T>(a, b);
      s_rho[j * kSmallLd + i] = small_pair<T>(a, i == j ? b : -b);
    }
    lds_barrier();
    own = s_rho[e];
  }
  if (in) {
    p.re[i * p.ld + j] = own[0];
    p.im[i * p.ld + j] = own[1];
  }
  if (tid == 0) {
    p.aux[0] = sc.sink;
    p.aux[1] = sc.rot;
    p.aux[2] = sc.lost;
    p.aux[3] = sc.steps;
    p.aux[4] = sc.scale;
  }
}

// Longer rows of dU, from the series of its exponential (series_tile.hpp) over
// H's few entries a row (D at most): both rotations in Horner form on one LDS
// array, along the rows and then along the columns, one barrier a term (v
// alternates between two arrays).
template <typename T, int D, int G, int NT>
__global__ __launch_bounds__(NT) void small_series_kernel(SmallArgs<T> p) {
  typedef T cplx __attribute__((ext_vector_type(2)));
  __shared__ cplx s_v[2][kSmallN * kSmallLd];
  __shared__ int32_t s_state[kSmallN], s_at[D][kSmallN];
  __shared__ T s_k[D][kSmallN];
  static_assert(D * kSmallN <= NT, "one entry per thread");
  const int n = p.n, tid = int(threadIdx.x), lane = tid & 63;
  const SmallSeries<T> &q = p.series;
  const int i = tid / n, j = tid - i * n;
  const bool in = i < n, low = in && j <= i;
  const int e = in ? i * kSmallLd + j : 0, ei = in ? i : 0, ej = in ? j : 0;
  // K's entries by state, through LDS (a thread's own reads of the tables cost
  // a call of one step 1 to 4 us); every load is issued before the first wait
  const int d0 = tid / kSmallN, slot = tid & (kSmallN - 1);
  const bool has = d0 < D && d0 < q.entries && slot < n;
  int32_t to = 0;
  T k = T(0);
  if (has) {
    to = q.entry_at[d0 * 64 + slot] >> __builtin_ctz(unsigned(q.slot_bytes));
    k = q.entry_val[d0 * 64 + slot];
  }
  if (tid < n) s_state[tid] = q.slot_col[tid];
  cplx x = small_pair<T>(0, 0);
  if (in) x = small_pair<T>(p.re[i * p.ld + j], p.im[i * p.ld + j]);
  const double aj = q.phase[2 * ej], bj = q.phase[2 * ej + 1], ai = q.phase[2 * ei],
               bi = -q.phase[2 * ei + 1];
  SmallElement<T, G> el;
  el.load(p, ei, ej, lane);
  SmallScalars sc{p.aux[0], p.aux[1], p.aux[2], p.aux[3], p.aux[4]};
  lds_barrier();
  if (d0 < D && slot < n) {
    s_at[d0][s_state[slot]] = has ? s_state[to] : 0;
    s_k[d0][s_state[slot]] = k;
  }
  lds_barrier();
  // K's rows j and i as neighbours along this element's row and column
  int at1[D], at2[D];
  T k1[D], k2[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    at1[d] = ei * kSmallLd + s_at[d][ej];
    at2[d] = s_at[d][ei] * kSmallLd + ej;
    k1[d] = s_k[d][ej];
    k2[d] = s_k[d][ei];
  }
  // the phase left over by the two shifts: e^{i (shift_j - shift_i) dt} - 1
  const double q_re = ai + aj + (ai * aj - bi * bj), q_im = bi + bj + (ai * bj + bi * aj);

  int flip = 0;
  // v <- x + ... ; returns d with (e^{sgn i K dt} x) = x + d
  auto rotate = [&](const cplx &own, const int (&at)[D], const T (&k)[D], T sgn) {
    cplx t;
    if (in) s_v[flip][e] = own;
    for (int m = q.order; m >= 1; --m) {
      lds_barrier();
      const cplx *v = s_v[flip];
      t = small_pair<T>(0, 0);
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const cplx g = v[at[d]];
        t[0] = fma(k[d], g[0], t[0]);
        t[1] = fma(k[d], g[1], t[1]);
      }
      const T w = sgn * T(q.ratio[m]);
      flip ^= 1;
      if (m == 1) return small_pair<T>(-w * t[1], w * t[0]);
      if (in) s_v[flip][e] = small_pair<T>(fma(-w, t[1], own[0]), fma(w, t[0], own[1]));
    }
    return t;
  };
  for (int64_t s = 0; s < p.steps; ++s) {
    // T = rho e^{i K dt} along the rows, Z = e^{-i K dt} T along the columns
    const cplx d1 = rotate(x, at1, k1, T(1));
    const cplx t = small_pair<T>(x[0] + d1[0], x[1] + d1[1]);
    const cplx d2 = rotate(t, at2, k2, T(-1));
    // z = (1 + q)(t + d2)
    const double yr = double(t[0]) + double(d2[0]), yi = double(t[1]) + double(d2[1]);
    const cplx z = small_pair<T>(T(double(t[0]) + (double(d2[0]) + (q_re * yr - q_im * yi))),
                                 T(double(t[1]) + (double(d2[1]) + (q_re * yi + q_im * yr))));
    // (the array that no wave reads any more)
    cplx *s_z = s_v[flip];
    if (low) s_z[e] = z;
    lds_barrier();
    const double zd = double(s_z[el.dw][0]);
    double xr, xi;
    el.decohere(z, s_z, xr, xi);
    sc.advance(p, el, zd);
    // rho' = scale * (Z + dt D(Z)) on and below the diagonal, mirrored
    flip ^= 1;
    cplx *s_x = s_v[flip];
    if (low) {
      const T a = T(xr * sc.scale), b = i == j ? T(0) : T(xi * sc.scale);
      s_x[e] = small_pair<T>(a, b);
      s_x[j * kSmallLd + i] = small_pair<T>(a, i == j ? b : -b);
    }
    lds_barrier();
    x = s_x[e];
    flip ^= 1;
  }
  if (in) {
    p.re[i * p.ld + j] = x[0];
    p.im[i * p.ld + j] = x[1];
  }
  if (tid == 0) {
    p.aux[0] = sc.sink;
    p.aux[1] = sc.rot;
    p.aux[2] = sc.lost;
    p.aux[3] = sc.steps;
    p.aux[4] = sc.scale;
  }
}

template <typename T, int NT>
static hipError_t launch_small_series(const SmallArgs<T> &a, hipStream_t s) {
  const dim3 one(1), threads(NT);
  if (a.series.entries <= 4) return launch_kernel(small_series_kernel<T, 4, 6, NT>, one, threads, 0, s, a);
  return launch_kernel(small_series_kernel<T, 8, 6, NT>, one, threads, 0, s, a);
}

template <typename T, int NT>
static hipError_t launch_small_rows(const SmallArgs<T> &a, hipStream_t s) {
  const dim3 one(1), threads(NT);
  if (a.n_gather <= 2) {
    if (a.row_max <= 2) return launch_kernel(small_rows_kernel<T, 2, 2, NT>, one, threads, 0, s, a);
    if (a.row_max <= 4) return launch_kernel(small_rows_kernel<T, 4, 2, NT>, one, threads, 0, s, a);
    return launch_kernel(small_rows_kernel<T, 8, 2, NT>, one, threads, 0, s, a);
  }
  if (a.row_max <= 4) return launch_kernel(small_rows_kernel<T, 4, 6, NT>, one, threads, 0, s, a);
  return launch_kernel(small_rows_kernel<T, 8, 6, NT>, one, threads, 0, s, a);
}

template <typename T>
hipError_t launch_small_steps(const SmallArgs<T> &a, hipStream_t s) {
  if (a.n < 1 || a.n > kSmallN || a.ld < a.n || a.steps < 0) return hipErrorInvalidValue;
  for (int64_t done = 0; done < a.steps; done += kSmallStepsPerLaunch) {
    SmallArgs<T> b = a;
    b.steps = std::min<int64_t>(kSmallStepsPerLaunch, a.steps - done);
    // up to eight entries in a row of dU: two sweeps over them against two per
    // term of the series (us per step, rows of dU / series: N = 18 with blocks of
    // two to eight states FP32 0.8 ... 1.0 / 1.4 ... 3.0, FP64 0.9 ... 1.2 / 2.5 ...
    // 3.4; N = 32, three channels, FP64 5.1 / 5.6); else the series while H's rows
    // have up to eight (N = 32 lattice 17.0 -> 2.7 us FP32, 16.6 -> 4.8 FP64; N =
    // 12 2.4 -> 1.2 and 2.0).  A call of one step takes about as long by either (N =
    // 18 FP32 7.8 / 6.9, FP64 8.2 / 8.1; 9.4 in the general kernel).
    hipError_t e;
    const bool series = a.n_gather <= 6 && a.series.order > 0 && a.series.entries <= 8;
    if (a.n_gather <= 6 && a.row_max <= 8)
      e = a.n <= 8 ? launch_small_rows<T, 64>(b, s)
          : a.n <= 16 ? launch_small_rows<T, 256>(b, s)
          : a.n <= 22 ? launch_small_rows<T, 512>(b, s) : launch_small_rows<T, 1024>(b, s);
    else if (series)
      e = a.n <= 16 ? launch_small_series<T, 256>(b, s)
          : a.n <= 22 ? launch_small_series<T, 512>(b, s) : launch_small_series<T, 1024>(b, s);
    else
      e = launch_kernel(small_steps_kernel<T>, dim3(1), dim3(kSmallThreads), 0, s, b);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template hipError_t launch_small_steps<float>(const SmallArgs<float> &, hipStream_t);
template hipError_t launch_small_steps<double>(const SmallArgs<double> &, hipStream_t);

}  // namespace qme
