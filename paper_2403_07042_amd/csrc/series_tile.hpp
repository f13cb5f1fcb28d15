// Row passes of the rotation rho_u = U rho U^dag with U = exp(-i H dt) applied
// by its Taylor series instead of as a dense matrix.
//
// H is sparse (a few couplings per state), so U v needs the series' few terms
// of a sparse product where the dense product needs N multiply-adds per
// element.  U is symmetric (H is real symmetric), so with
//   R(X) = X conj(U)          (each row x of X by itself: conj(U) x)
// the rotation is two row passes with a conjugate transpose between:
//   W = R(rho),  rho_u = R(W^dag)   (= W^dag U^dag = U rho^dag U^dag),
// the first pass writing W^dag.  Both passes read whole rows (contiguous).
//
// One workgroup takes R rows.  The rows' elements at one basis state form one
// unit of 16 (or 8) bytes per plane, so a lane gathers a neighbouring state of
// all its rows with one LDS read per plane.  The series runs in Horner form
//   v <- x + (A v) / k,  k = order .. 2,   delta = A v,   result = x + delta,
// A = +-i K dt with K = H less a shift that is constant on each connected
// component of H (it commutes with H; where the shifts differ, e^{-+i shift dt} - 1
// is formed in FP64 by the plan and applied at the end in the storage type, as a
// small term).  v lives in LDS, x and the sums in registers: a term is one gather
// sweep and two barriers.  (The coefficients are those of the series economised
// on |K dt| <= theta, which needs a term or two less: ratio[k] stands for 1 / k.)
// The result is x + (small terms): the terms are summed in the storage type and the
// last addition rounds once -- in the storage type, or in FP64 with the decoherence
// factor where a step is folded.
//
// What bounds it: at N = 2048 a pass moves 33.5 MB in and 33.5 MB out (a copy of
// that size takes 8.4 us) and reads 0.4 GB of LDS per rotation; its loads, terms
// and stores run one after another in a workgroup, and the launch is one round
// of them.  Measured there: 21 + 20 us FP32 (three terms) and 48 + 48 us FP64
// (four), against 387 + 224 and 844 + 452 us of the dense products; a folded
// step in one pass (kSeriesStep) 32.8 us FP32 and 83.7 us FP64.  The rest of
// the range with series as short, two passes / one: N = 100 9.0 / 5.8 us FP32 and
// 13.3 / 7.4 FP64, 500 15.1 / 8.4 and 19.5 / 12.8, 1024 21.4 / 13.6 and 36.7 / 26.7,
// 4096 161 / 152 and 611 / 540.  Longer series and rows, and N past 4096:
// series_step_us and series_one_pass (series.hip).
// The registers (128 at four waves per SIMD) do not hold every shape: bytes of
// scratch per lane in the two passes / in kSeriesStep are none / 96 (FP32) and 112
// (FP64) at N = 1025 ... 2048, 0 to 20 / 124 and 20 to 48 / 152 up to 4096, 120 to
// 148 / 280 and 132 to 156 / 304 up to 5120, 164 to 240 / about 305 past it.  There
// the spilled part of the rows makes the way through memory as well.
#pragma once

#include <cstdint>

#include "device.hpp"
#include "dissipate_tile.hpp"
#include "lds_barrier.hpp"

namespace qme {

// Workgroups are dealt to the XCDs round-robin.  Consecutive row groups go to
// one XCD, so the R-element pieces of a line that the transposed writes leave
// meet in that XCD's L2.
__device__ __forceinline__ int series_group(int block, int groups) {
  const int per = (groups + 7) >> 3;
  return (block & 7) * per + (block >> 3);
}

// A value that every lane of the wave holds, kept in scalar registers.
__device__ __forceinline__ double series_uniform(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_readfirstlane(int(b)), hi = __builtin_amdgcn_readfirstlane(int(b >> 32));
  return __builtin_bit_cast(double, (static_cast<long long>(hi) << 32) | unsigned(lo));
}

template <typename T>
__device__ __forceinline__ T series_fma(T a, T b, T c) {
  if constexpr (sizeof(T) == 4) return __builtin_fmaf(a, b, c);
  else return __builtin_fma(a, b, c);
}

// W^dag between the two passes: element (c, r) in slot order, units of R
// consecutive r of one c, the units of four c side by side and then the next
// group of R r.  The first pass's workgroup (one group of R r, every c) writes,
// and the second's (R of the c, every r) reads, whole pieces of four units (64
// or 128 bytes).  A transposed row-major plane had it write single 16-byte
// units, one request of the L2 each: 13 of the 31 us that the first pass took
// at N = 2048.
__device__ __forceinline__ int64_t series_unit(int c, int g, int groups) {
  return (int64_t(c >> 2) * groups + g) * 4 + (c & 3);
}

// MODE kSeriesFirst: reads the state, writes W^dag in blocks (series_unit).
// MODE kSeriesBoth: as kSeriesFirst, and writes W's own rows too.
// MODE kSeriesLower: reads those blocks, writes the rows of rho_u on and below
// the diagonal.
// MODE kSeriesFold: as kSeriesLower with the decoherence factor applied, whole
// rows written, the diagonal before the decoherence kept for the trace
// (CgemmArgs::fold_d).  Both triangles come from their own rows here, so they
// agree to rounding only; the closing pass of the call restores the exact
// symmetry (Herm commutes with every step).
// MODE kSeriesStep: kSeriesFold and the next step's kSeriesFirst in one: a row
// of the state is all that its own next pass needs, so it stays in the
// registers (but for what the shape spills) and only the blocks pass through
// memory, once per step.
//
// The renormalisation factor is a scalar: it stays pending (DissArgs::pend)
// until the call's closing pass.  Factors near one are applied as x + (small
// terms), the small terms and their coefficients in the storage type, so that a
// result is rounded once, at the last addition.
template <typename T, int R, int S, int NT, int MODE>
__device__ __forceinline__ void series_rows(const SeriesArgs<T> &a, int group, unsigned char *lds) {
  // (a batch's passes give each instance the bits of its own passes: the
  // arithmetic must not depend on what the compiler fuses in each shape)
#pragma clang fp contract(off)
  typedef T unit __attribute__((ext_vector_type(R)));
  constexpr bool kReadRows = MODE == kSeriesFirst || MODE == kSeriesBoth;
  constexpr bool kBlocks = kReadRows || MODE == kSeriesStep;    // writes blocks
  constexpr bool kRows = MODE == kSeriesLower || MODE == kSeriesFold || MODE == kSeriesBoth;   // writes rows
  // v in LDS: a unit's 16-byte parts (one or two) in planes of their own, so
  // that lanes with neighbouring slots read without bank conflicts; the
  // imaginary planes follow the real ones
  constexpr int kPart = sizeof(unit) < 16 ? int(sizeof(unit)) : 16;
  constexpr int P = int(sizeof(unit)) / kPart;
  constexpr int E = R / P;
  typedef T part __attribute__((ext_vector_type(E)));
  constexpr int kPlane = S * NT * kPart;
  auto put = [](unsigned char *base, int slot, const unit &re, const unit &im) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      part a, b;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        a[e] = re[p * E + e];
        b[e] = im[p * E + e];
      }
      *reinterpret_cast<part *>(base + p * kPlane + slot * kPart) = a;
      *reinterpret_cast<part *>(base + (P + p) * kPlane + slot * kPart) = b;
    }
  };
  const int tid = int(threadIdx.x);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = int(a.n);
  const int slots = (n + 63) & ~63;
  const int groups = (n + R - 1) / R;
  const int q0 = group * R;            // the rows: states of slots q0 .. q0 + R - 1
  int row[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    row[r] = __builtin_amdgcn_readfirstlane(a.slot_col[min(q0 + r, n - 1)]);

  // Wave w takes slices w S .. w S + S - 1 of 64 slots.  With one or two
  // slices a wave keeps their first C entries in registers for all terms;
  // with more it loads a slice's first C when the slice before it has used
  // its own.  Further entries are loaded as they come.
  constexpr int C = sizeof(T) == 4 ? 4 : 3;
  constexpr int B = S <= 2 ? S : 1;
  int off[S + 1];
#pragma unroll
  for (int s = 0; s <= S; ++s) off[s] = a.slice_off[min(wave * S + s, slots >> 6)];
  struct Entries {
    int32_t at[C];
    T val[C];
  };
  Entries buf[B];
  auto fetch = [&](Entries &to, int first) {
    const int32_t *p = a.entry_at + int64_t(first) * 64;
    const T *q = a.entry_val + int64_t(first) * 64;
#pragma unroll
    for (int i = 0; i < C; ++i) {
      to.at[i] = p[unsigned(i * 64 + lane)];
      to.val[i] = q[unsigned(i * 64 + lane)];
    }
  };
  auto fetch_first = [&]() {
#pragma unroll
    for (int s = 0; s < B; ++s) fetch(buf[s], off[s]);
  };
  fetch_first();

  // the rows, one state per lane.  A slot or row past the end repeats the
  // last one: no entry reads it and it is not written.
  unit x_re[S], x_im[S];
  unsigned col[S];
#pragma unroll
  for (int s = 0; s < S; ++s) col[s] = unsigned(a.slot_col[unsigned(min((wave * S + s) * 64 + lane, n - 1))]);
  if constexpr (kReadRows) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const T *p_re = a.x_re + int64_t(row[r]) * a.ld, *p_im = a.x_im + int64_t(row[r]) * a.ld;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        x_re[s][r] = p_re[col[s]];
        x_im[s][r] = p_im[col[s]];
      }
    }
  } else {
    unsigned at[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int slot = min((wave * S + s) * 64 + lane, n - 1);
      at[s] = unsigned(series_unit(0, slot / R, groups)) * R + unsigned(slot % R);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t o = series_unit(min(q0 + r, n - 1), 0, groups) * R;
      const T *p_re = a.x_re + o, *p_im = a.x_im + o;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        x_re[s][r] = p_re[at[s]];
        x_im[s][r] = p_im[at[s]];
      }
    }
  }
  unit t_re[S], t_im[S];
  const T sgn = T(a.sign), w1 = sgn * T(a.ratio[1]);
  // the terms of x's rows, up to delta = (+-i w1 t)
  auto rotate = [&]() {
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int slot = (wave * S + s) * 64 + lane;
    put(lds, slot, x_re[s], x_im[s]);
  }

  for (int k = a.order; k >= 1; --k) {
    lds_barrier();
#pragma unroll
    for (int s = 0; s < S; ++s) {
#pragma unroll
      for (int r = 0; r < R; ++r) t_re[s][r] = t_im[s][r] = T(0);
      auto add = [&](T val, int at) {
        // (planes beyond the reach of a read's offset: their addresses formed
        // here, not kept for every entry and term)
        if constexpr ((2 * P - 1) * kPlane > 65535) asm volatile("" : "+v"(at));
#pragma unroll
        for (int p = 0; p < P; ++p) {
          const part g_re = *reinterpret_cast<const part *>(lds + at + p * kPlane);
          const part g_im = *reinterpret_cast<const part *>(lds + at + (P + p) * kPlane);
#pragma unroll
          for (int e = 0; e < E; ++e) {
            t_re[s][p * E + e] = series_fma<T>(val, g_re[e], t_re[s][p * E + e]);
            t_im[s][p * E + e] = series_fma<T>(val, g_im[e], t_im[s][p * E + e]);
          }
        }
      };
      auto chunk = [&](const Entries &q, int cnt) {
#pragma unroll
        for (int i = 0; i < C; ++i)
          if (i < cnt) add(q.val[i], q.at[i]);
      };
      const int cnt = off[s + 1] - off[s];
      Entries &own = buf[s % B];
      const int next = off[(s + 1) % S];
      chunk(own, cnt);
      if constexpr (S <= 2) {
        for (int e = C; e < cnt; e += C) {
          Entries more;
          fetch(more, off[s] + e);
          chunk(more, cnt - e);
        }
      } else {
        for (int e = C; e < cnt; e += C) {
          fetch(own, off[s] + e);
          chunk(own, cnt - e);
        }
        fetch(own, next);
      }
    }
    if (k == 1) break;
    lds_barrier();
    const T w = sgn * T(a.ratio[k]);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      unit n_re, n_im;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        n_re[r] = series_fma<T>(-w, t_im[s][r], x_re[s][r]);
        n_im[r] = series_fma<T>(w, t_re[s][r], x_im[s][r]);
      }
      const int slot = (wave * S + s) * 64 + lane;
      put(lds, slot, n_re, n_im);
    }
  }
  };
  // t <- d, the small part of the result x + d
  auto finish = [&]() {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const unit was = t_re[s];
      t_re[s] = -w1 * t_im[s];
      t_im[s] = w1 * was;
    }
    if (a.phase) {   // (1 + q)(x + d)
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const T q_re = T(a.phase[2 * col[s]]), q_im = sgn * T(a.phase[2 * col[s] + 1]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const T yr = x_re[s][r] + t_re[s][r], yi = x_im[s][r] + t_im[s][r];
          t_re[s][r] = series_fma<T>(-q_im, yi, series_fma<T>(q_re, yr, t_re[s][r]));
          t_im[s][r] = series_fma<T>(q_im, yr, series_fma<T>(q_re, yi, t_im[s][r]));
        }
      }
    }
  };

  auto decohere = [&]() {
    // x <- the decoherence step of the rotated rows
    double row_d[R];
#pragma unroll
    for (int r = 0; r < R; ++r)
      row_d[r] = series_uniform(-0.5 * a.fold_dt * a.fold_d[row[r]]);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const double col_d = -0.5 * a.fold_dt * a.fold_d[col[s]];
      // (the trace is taken of the diagonal as it is stored)
      T diag = T(0);
      bool own = false;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const bool here = unsigned(row[r]) == col[s] && q0 + r < n;
        own = own || here;
        diag = here ? x_re[s][r] + t_re[s][r] : diag;
      }
      if (own && (wave * S + s) * 64 + lane < n) a.zdiag[col[s]] = double(diag);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double f = row_d[r] + col_d;
        const double zr = double(x_re[s][r]) + double(t_re[s][r]);
        const double zi = double(x_im[s][r]) + double(t_im[s][r]);
        x_re[s][r] = T(__builtin_fma(f, zr, zr));
        x_im[s][r] = T(__builtin_fma(f, zi, zi));
      }
    }
  };

  rotate();
  finish();
  if constexpr (MODE == kSeriesFold || MODE == kSeriesStep) decohere();
  if constexpr (MODE == kSeriesStep) {
    fetch_first();
    lds_barrier();   // every wave has read v
    rotate();
    finish();
  }
  // (the row passes hand their results to LDS, by state, so that the rows are
  // written in order: the slots' order would leave parts of lines)
  if constexpr (kRows) lds_barrier();
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const int slot = (wave * S + s) * 64 + lane;
    if (slot >= n) continue;
    const unsigned c = col[s];
    unit w_re = x_re[s], w_im = x_im[s];
    if constexpr (MODE != kSeriesFold) {
      w_re += t_re[s];
      w_im += t_im[s];
    }
    if constexpr (kBlocks) {
      const int64_t u = series_unit(0, group, groups);
      const unsigned o = unsigned(series_unit(slot, 0, groups));
      (reinterpret_cast<unit *>(a.o_re) + u)[o] = w_re;
      (reinterpret_cast<unit *>(a.o_im) + u)[o] = -w_im;
    }
    if constexpr (kRows) put(lds, int(c), w_re, w_im);
  }
  if constexpr (kRows) {
    lds_barrier();
    unit w_re[S], w_im[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const part a_re = *reinterpret_cast<const part *>(lds + (s * NT + tid) * kPart + p * kPlane);
        const part a_im = *reinterpret_cast<const part *>(lds + (s * NT + tid) * kPart + (P + p) * kPlane);
#pragma unroll
        for (int e = 0; e < E; ++e) {
          w_re[s][p * E + e] = a_re[e];
          w_im[s][p * E + e] = a_im[e];
        }
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (q0 + r >= n) break;
      T *p_re = (kBlocks ? a.r_re : a.o_re) + int64_t(row[r]) * a.ld;
      T *p_im = (kBlocks ? a.r_im : a.o_im) + int64_t(row[r]) * a.ld;
      const int end = MODE == kSeriesLower ? row[r] + 1 : n;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const unsigned c = unsigned(s * NT + tid);
        if (int(c) < end) {
          p_re[c] = w_re[s][r];
          p_im[c] = w_im[s][r];
        }
      }
    }
  }
}

}  // namespace qme
