// Launchers of the series row passes (series_tile.hpp).
#include "series_tile.hpp"

#include <algorithm>
#include <cmath>

#include "ctx.hpp"

namespace qme {

// as the trace pass, so that the factor is bitwise the same
static constexpr int kSeriesTraceThreads = 256;

// A pass may also form an earlier step's trace, in one further workgroup that
// runs beside the others (tr_zdiag).
template <typename T, int R, int S, int NT, int MODE>
__global__ __launch_bounds__(NT, 4) void series_pass_kernel(SeriesArgs<T> a) {
  extern __shared__ __align__(16) unsigned char lds[];
  if (a.tr_zdiag && blockIdx.x == gridDim.x - 1) {
    DissArgs<T> d{};
    d.n = a.n;
    d.dt = a.tr_dt;
    d.trw = a.tr_w;
    d.leak = a.tr_leak;
    d.zdiag = a.tr_zdiag;
    d.aux_in = d.aux_out = a.tr_aux;
    d.pend = a.tr_pend;
    double *st = reinterpret_cast<double *>(lds);
    constexpr int W = kSeriesTraceThreads / 64;
    trace_body<T, kSeriesTraceThreads, true>(d, st, st + W, st + 2 * W);
    return;
  }
  const int group = series_group(int(blockIdx.x), a.groups);
  if (group >= a.groups) return;
  series_rows<T, R, S, NT, MODE>(a, group, lds);
}

// The closing pass of a call of folded series steps: X *= factor (FP64) with
// the upper triangle taken from the lower, so the stored state is exactly
// Hermitian.  One workgroup per 32 x 32 tile on or below the diagonal, its
// mirror staged through LDS (32 x 33 elements).
template <typename T>
__global__ __launch_bounds__(256) void series_close_kernel(T *re, T *im, int64_t ld, int64_t n,
                                                           const double *factor) {
  __shared__ T s_re[32][33], s_im[32][33];
  int bi = int((sqrtf(8.0f * float(blockIdx.x) + 1.0f) - 1.0f) * 0.5f);
  while ((bi + 1) * (bi + 2) / 2 <= int(blockIdx.x)) ++bi;
  while (bi * (bi + 1) / 2 > int(blockIdx.x)) --bi;
  const int bj = int(blockIdx.x) - bi * (bi + 1) / 2;
  const double f = *factor;
  const int c = int(threadIdx.x) & 31, r0 = int(threadIdx.x) >> 5;
  T x_re[4], x_im[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t u = std::min<int64_t>(int64_t(bi) * 32 + r0 + 8 * i, n - 1);
    const int64_t v = std::min<int64_t>(int64_t(bj) * 32 + c, n - 1);
    x_re[i] = re[u * ld + v];
    x_im[i] = im[u * ld + v];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + 8 * i;
    const int64_t u = int64_t(bi) * 32 + r, v = int64_t(bj) * 32 + c;
    const T a = T(f * double(x_re[i])), b = u == v ? T(0) : T(f * double(x_im[i]));
    s_re[r][c] = a;
    s_im[r][c] = b;
    if (u < n && v <= u) {
      re[u * ld + v] = a;
      im[u * ld + v] = b;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + 8 * i;   // row of the mirror: a column of the tile
    const int64_t u = int64_t(bj) * 32 + r, v = int64_t(bi) * 32 + c;
    if (v < n && u < v) {
      re[u * ld + v] = s_re[c][r];
      im[u * ld + v] = -s_im[c][r];
    }
  }
}

namespace {

template <typename T, int R, int S, int NT, int MODE>
hipError_t launch_one(const SeriesArgs<T> &in, hipStream_t s) {
  SeriesArgs<T> a = in;
  a.groups = int32_t((a.n + R - 1) / R);
  constexpr size_t lds = size_t(2) * S * NT * R * sizeof(T);   // up to all 160 KB
  const auto kernel = series_pass_kernel<T, R, S, NT, MODE>;
  if (lds > 48 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
  }
  const unsigned grid = unsigned((a.groups + 7) / 8 * 8) + (a.tr_zdiag ? 1 : 0);
  return launch_kernel(kernel, dim3(grid), dim3(NT), uint32_t(lds), s, a);
}

template <typename T, int R, int S, int NT>
hipError_t launch_mode(const SeriesArgs<T> &a, int mode, hipStream_t s) {
  switch (mode) {
    case kSeriesFirst: return launch_one<T, R, S, NT, kSeriesFirst>(a, s);
    case kSeriesLower: return launch_one<T, R, S, NT, kSeriesLower>(a, s);
    case kSeriesFold: return launch_one<T, R, S, NT, kSeriesFold>(a, s);
    case kSeriesStep: return launch_one<T, R, S, NT, kSeriesStep>(a, s);
    case kSeriesBoth: return launch_one<T, R, S, NT, kSeriesBoth>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// The shape of a pass: bytes of a unit, slices per wave, threads.  A workgroup
// holds its rows in LDS (2 x 64 states x slices x waves x bytes: up to all of
// 160 KB) and in registers (128 at four waves per SIMD), so the rows get fewer
// as N grows.
struct SeriesShape {
  int bytes, slices, threads;
};
static SeriesShape series_shape(int64_t n) {
  if (n <= 256) return {16, 1, 256};
  if (n <= 512) return {16, 2, 256};
  if (n <= 1024) return {16, 2, 512};
  if (n <= 2048) return {32, 2, 1024};
  if (n <= 4096) return {16, 4, 1024};
  if (n <= 5120) return {16, 5, 1024};
  return {8, 8, 1024};
}

int series_slot_bytes(int64_t n) { return std::min(series_shape(n).bytes, 16); }
int series_slices_per_wave(int64_t n) { return series_shape(n).slices; }

// A folded step in one pass saves a round trip of the state, but past N = 4096 its
// body holds more than the registers (101 of them spilled per lane at five slices
// per wave, 112 and more at eight), so that a long series makes up for the round
// trip.  Measured (us per step, one pass / two, four couplings per state): FP32 N
// = 4131 order 3 294 / 284, 5 374 / 344, 7 454 / 405, 10 573 / 495; 5120 order 3 342
// / 350, 5 421 / 409; 6000 order 5 1109 / 1127, 7 1365 / 1327, 10 1744 / 1648; FP64 N =
// 4131 order 10 1764 / 1749 and 5120 2211 / 2256; 6000 order 4 3072 / 3069, 5 3647 /
// 3575, 10 7140 / 6656.  Up to N = 4096 one pass is the faster or equal (2048 FP32
// 36 / 43, 4096 order 7 251 / 255).
bool series_one_pass(int64_t n, int elem, int order) {
  if (n <= 4096) return true;
  if (elem == 8) return n <= 5120 || order < 5;
  return order < (n <= 5120 ? 5 : 7);
}

// A step is as slow as the longest wave of a workgroup, or as the workgroup's
// LDS reads where all its rows are long, times the rounds of workgroups on the
// device: not as the mean row of H.  The figures are fits to steps timed on the
// MI355X with rows of 2 to 400 entries and with a star (one state coupled to all
// others) at N = 40 ... 8190, in FP32 and FP64 (order 8 and 12); of 380 pairs of
// times six choices cost more than 5% against the better form (at most 28%).
// Entries: a wave takes them C at a time, the first C of a slice (of the shapes
// with one or two slices) from registers, each further C after a load that is
// waited for (0.42 us FP32, 0.31 FP64; four slices and more in FP64 0.5, eight
// 0.8).  Series / dense, us per step: star N = 65 103 / 14, 501 805 / 36, 2048
// 3463 / 615; rows of 64 at N = 513 217 / 43, 1025 260 / 144, 2048 407 / 643,
// 4096 1823 / 4717; rows of 128 at N = 2048 852 / 646; of 200 at 4096 6797 / 4740.
// LDS: 128 bytes per clock, half as much again where lanes read scattered states
// (bank conflicts: random rows of 32 at N = 2048 371 against 201).
double series_step_us(const SeriesPlan &p, int64_t n, int elem, bool folded, int cus) {
  const SeriesShape f = series_shape(n);
  const int c = elem == 4 ? 4 : 3;
  const double load = f.slices == 8 ? 0.8 : elem == 4 ? 0.42 : f.slices <= 2 ? 0.31 : 0.5;
  const int64_t slices = int64_t(p.slice_off.size()) - 1;
  double longest = 0.0;
  for (int64_t q0 = 0; q0 < slices; q0 += f.slices) {
    double wave = 0.0;
    for (int64_t q = q0; q < std::min(slices, q0 + f.slices); ++q) {
      const int len = p.slice_off[size_t(q) + 1] - p.slice_off[size_t(q)];
      const double kept = f.slices <= 2 && len > 0 ? 1.0 : 0.0;
      wave += 0.15 * kept + load * std::max(0.0, double(len) / c - kept);
    }
    longest = std::max(longest, wave);
  }
  // workgroups that a compute unit holds (LDS, 1024 threads at four waves per
  // SIMD), and the rounds that the row groups need
  const int per_cu = std::min(163840 / (2 * f.slices * f.threads * f.bytes), 1024 / f.threads);
  const int64_t groups = (n * elem + f.bytes - 1) / f.bytes, room = int64_t(cus) * per_cu;
  const double rounds = double((groups + room - 1) / room);
  const double resident = double(std::min<int64_t>(per_cu, (groups + cus - 1) / cus));
  const double lds = resident * double(p.slice_off.back()) * 64.0 * 2.0 * f.bytes / (137.0 * 2400.0) *
                     (1.0 + 0.55 * p.scattered);
  const double term = (f.threads == 1024 ? 1.8 : elem == 4 ? 0.4 : 0.3) + std::max(longest, lds);
  const double move = 4.0 * double(n) * double(n) * elem / 5e6;   // the planes in and out, 5 TB/s
  return rounds * 2.0 * p.order * term + move + 2.0 + (folded ? 0.0 : 6.0 + move);
}

// Measured steps by dense products (MI355X, us per step; the launches' latency
// up to N = 256, the matrix cores from N = 1024), between them in proportion of
// the logarithms.
double dense_step_us(int precision, int64_t n) {
  static constexpr double kN[7] = {64, 128, 256, 512, 1024, 2048, 4096};
  static constexpr double kFp64[7] = {21, 22.5, 30, 68, 245, 1310, 10500};
  static constexpr double kFp32[7] = {14, 17, 26, 43, 140, 620, 4650};
  static constexpr double kBf16x3[7] = {23, 24.5, 29, 42, 150, 420, 4050};
  const double *us = precision == QME_FP64 ? kFp64 : precision == QME_FP32 ? kFp32 : kBf16x3;
  return interpolate_us(kN, us, 7, 3.0, double(n));
}

double interpolate_us(const double *at, const double *us, int count, double power, double n) {
  if (n <= at[0]) return us[0];
  for (int i = 1; i < count; ++i)
    if (n <= at[i])
      return us[i - 1] * std::pow(us[i] / us[i - 1], std::log(n / at[i - 1]) / std::log(at[i] / at[i - 1]));
  return us[count - 1] * std::pow(n / at[count - 1], power);
}

template <typename T>
hipError_t launch_series_pass(const SeriesArgs<T> &a, int mode, hipStream_t s) {
  constexpr int E = int(sizeof(T));
  if (a.n < 1 || a.n > kSeriesMaxN || a.ld < a.n || a.order < 1 || a.order > kSeriesMaxOrder)
    return hipErrorInvalidValue;
  const SeriesShape f = series_shape(a.n);
  // (W^dag takes whole blocks of four units by R)
  if ((a.n + 3) / 4 * 4 * ((a.n * E + f.bytes - 1) / f.bytes) * (f.bytes / E) > a.ld * a.ld)
    return hipErrorInvalidValue;
  if (f.bytes == 32) return launch_mode<T, 32 / E, 2, 1024>(a, mode, s);
  if (f.bytes == 8) return launch_mode<T, 8 / E, 8, 1024>(a, mode, s);
  if (f.slices == 1) return launch_mode<T, 16 / E, 1, 256>(a, mode, s);
  if (f.slices == 2 && f.threads == 256) return launch_mode<T, 16 / E, 2, 256>(a, mode, s);
  if (f.slices == 2) return launch_mode<T, 16 / E, 2, 512>(a, mode, s);
  if (f.slices == 4) return launch_mode<T, 16 / E, 4, 1024>(a, mode, s);
  return launch_mode<T, 16 / E, 5, 1024>(a, mode, s);
}

template <typename T>
hipError_t launch_series_close(T *re, T *im, int64_t ld, int64_t n, const double *factor, hipStream_t s) {
  const int64_t t = (n + 31) / 32;
  return launch_kernel(series_close_kernel<T>, dim3(unsigned(t * (t + 1) / 2)), dim3(256), 0, s, re, im,
                       ld, n, factor);
}

template hipError_t launch_series_close<float>(float *, float *, int64_t, int64_t, const double *, hipStream_t);
template hipError_t launch_series_close<double>(double *, double *, int64_t, int64_t, const double *, hipStream_t);
template hipError_t launch_series_pass<float>(const SeriesArgs<float> &, int, hipStream_t);
template hipError_t launch_series_pass<double>(const SeriesArgs<double> &, int, hipStream_t);

}  // namespace qme
