// Discrete Fourier transforms of real n^3 lattices, device side: mixed-radix
// line transforms in LDS, shared by the spectra, the vacuum initial state
// and the linearized integrator.
//
// A real field's transform F_k = sum_x f_x exp(-2 pi i k.x/n) has
// F_{-k} = conj F_k, so only kx = 0 .. n/2 is kept: half the modes, half the
// memory traffic and half the arithmetic of a complex transform.  The three
// axis passes are
//   x:    two real rows y, y + 1 form the complex row f_y + i f_{y+1}, whose
//         transform Z separates into theirs, A_k = (Z_k + conj Z_{n-k})/2 and
//         B_k = (Z_k - conj Z_{n-k})/2i;
//   y, z: complex columns, in place.
// The inverse runs them backwards.  What a caller does with a field before
// the first pass (drift, remainder) or with a mode after the last one
// (binning) is a functor of the pass, so no pass over memory is spent on it.
//
// Layout of the half spectrum: plane z, row y, mode kx at
// (z n + y) nhp + kx, nhp = n/2 + 1 rounded up to 8 for n >= 32 so that a
// group of 8 or more neighbouring columns is whole 128-byte lines.
//
// A workgroup transforms L lines of n values at once (L n <= 8 per thread)
// with Stockham stages of radix 8, 4, 2, 3, 5, 7 (and a direct sum for other
// prime factors): stage with Ns = product of the earlier radices reads
// x[j + q n/R], multiplies by exp(-2 pi i q (j mod Ns) / (Ns R)), transforms
// the R values and writes them at (j / Ns) Ns R + (j mod Ns) + q Ns, so the
// last stage leaves natural order.  Values pass from thread to thread through
// one LDS buffer; the first stage reads and the last one writes memory
// directly.  It is bound by memory: three passes over 8 n^3 bytes.  256^3 in
// FP64: x pass 73 us from a field and its drift (5.5 TB/s), 55 us from momenta,
// y pass 49 us (5.6 TB/s), four workgroups to a CU; one complex axis pass of a
// radix-2 transform with a barrier per factor 2 took 266 us, and a direct sum
// 52 us per axis at 96^3 (now 13 + 8 us).  Loads stay free of branches: with
// one around the second row of a pair and one around the field of a momentum
// the x passes took 118 and 78 us.
#pragma once

#include "device.h"

namespace symlat {

// 16-byte LDS elements, one of padding after every 8: the strided writes of a
// stage (R n_s apart) then spread over the banks.
__device__ __forceinline__ int lds_pad(int i) { return i + (i >> 3); }

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// -i a
__device__ __forceinline__ double2 cmi(double2 a) { return make_double2(a.y, -a.x); }

// Forward transforms of R values in registers (natural order in and out).
__device__ __forceinline__ void dft_r(double2 (&v)[2]) {
  const double2 a = v[0];
  v[0] = cadd(a, v[1]);
  v[1] = csub(a, v[1]);
}

__device__ __forceinline__ void dft_r(double2 (&v)[3]) {
  constexpr double s3 = 0.86602540378443864676;  // sin(2 pi/3)
  const double2 t = cadd(v[1], v[2]), d = csub(v[1], v[2]);
  const double2 m = make_double2(v[0].x - 0.5 * t.x, v[0].y - 0.5 * t.y);
  v[0] = cadd(v[0], t);
  // m -+ i s3 d
  v[1] = make_double2(m.x + s3 * d.y, m.y - s3 * d.x);
  v[2] = make_double2(m.x - s3 * d.y, m.y + s3 * d.x);
}

__device__ __forceinline__ void dft_r(double2 (&v)[4]) {
  const double2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]);
  const double2 c = cadd(v[1], v[3]), d = cmi(csub(v[1], v[3]));
  v[0] = cadd(a, c);
  v[1] = cadd(b, d);
  v[2] = csub(a, c);
  v[3] = csub(b, d);
}

// Odd prime R by symmetric pairs: with t_q = v_q + v_{R-q}, d_q = v_q -
// v_{R-q}, V_k = v_0 + sum_q cos(2 pi k q/R) t_q - i sum_q sin(2 pi k q/R) d_q.
template <int R>
__device__ __forceinline__ void dft_odd(double2 (&v)[R], const double (&cs)[R], const double (&sn)[R]) {
  constexpr int H = (R - 1) / 2;
  double2 t[H], d[H], out[R];
#pragma unroll
  for (int q = 0; q < H; ++q) {
    t[q] = cadd(v[q + 1], v[R - 1 - q]);
    d[q] = csub(v[q + 1], v[R - 1 - q]);
  }
  out[0] = v[0];
#pragma unroll
  for (int q = 0; q < H; ++q) out[0] = cadd(out[0], t[q]);
#pragma unroll
  for (int k = 1; k <= H; ++k) {
    double2 e = v[0], o = make_double2(0.0, 0.0);
#pragma unroll
    for (int q = 1; q <= H; ++q) {
      e.x += cs[(k * q) % R] * t[q - 1].x;
      e.y += cs[(k * q) % R] * t[q - 1].y;
      o.x += sn[(k * q) % R] * d[q - 1].x;
      o.y += sn[(k * q) % R] * d[q - 1].y;
    }
    out[k] = make_double2(e.x + o.y, e.y - o.x);
    out[R - k] = make_double2(e.x - o.y, e.y + o.x);
  }
#pragma unroll
  for (int k = 0; k < R; ++k) v[k] = out[k];
}

__device__ __forceinline__ void dft_r(double2 (&v)[5]) {
  constexpr double c1 = 0.30901699437494742410, c2 = -0.80901699437494742410;  // cos(2 pi k/5)
  constexpr double s1 = 0.95105651629515357212, s2 = 0.58778525229247312917;   // sin(2 pi k/5)
  constexpr double cs[5] = {1.0, c1, c2, c2, c1}, sn[5] = {0.0, s1, s2, -s2, -s1};
  dft_odd<5>(v, cs, sn);
}

__device__ __forceinline__ void dft_r(double2 (&v)[7]) {
  constexpr double c1 = 0.62348980185873353053, c2 = -0.22252093395631440429,
                   c3 = -0.90096886790241912624;  // cos(2 pi k/7)
  constexpr double s1 = 0.78183148246802980871, s2 = 0.97492791218182360702,
                   s3 = 0.43388373911755812048;   // sin(2 pi k/7)
  constexpr double cs[7] = {1.0, c1, c2, c3, c3, c2, c1}, sn[7] = {0.0, s1, s2, s3, -s3, -s2, -s1};
  dft_odd<7>(v, cs, sn);
}

__device__ __forceinline__ void dft_r(double2 (&v)[8]) {
  constexpr double h = 0.70710678118654752440;  // cos(pi/4)
  double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
  dft_r(e);
  dft_r(o);
  // o_k exp(-i pi k/4)
  o[1] = make_double2(h * (o[1].x + o[1].y), h * (o[1].y - o[1].x));
  o[2] = cmi(o[2]);
  o[3] = make_double2(h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y));
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[k] = cadd(e[k], o[k]);
    v[k + 4] = csub(e[k], o[k]);
  }
}

// How the values of a group of lines sit in LDS and how threads share them.
// Rows (the x axis, contiguous in memory): neighbouring threads take
// neighbouring elements of a line.
struct RowMap {
  int n;
  __device__ __forceinline__ int at(int l, int e) const { return lds_pad(l * n + e); }
  // butterfly b of nr per line -> (line, index)
  __device__ __forceinline__ void split(int b, int nr, unsigned m_nr, int& l, int& j) const {
    l = div_magic(b, m_nr);
    j = b - l * nr;
  }
};
// Columns (the y and z axes): neighbouring threads take neighbouring lines,
// whose values are neighbours in memory.
struct ColMap {
  int lg;  // log2 of the lines in a group
  __device__ __forceinline__ int at(int l, int e) const { return lds_pad((e << lg) | l); }
  __device__ __forceinline__ void split(int b, int, unsigned, int& l, int& j) const {
    l = b & ((1 << lg) - 1);
    j = b >> lg;
  }
};


// This thread's index, opaque to the optimiser: the addresses of every stage
// are cheap to form but many, and kept across a loop over groups of lines
// they took 250 registers (spilled at three wavefronts per SIMD).
__device__ __forceinline__ int fresh_tid() {
  int t = int(threadIdx.x);
  asm volatile("" : "+v"(t));
  return t;
}

// One stage of radix R over `lines` lines.  SYNC: the values are read from
// and written to the same LDS buffer, so all reads come before any write.
template <int NT, int R, bool SYNC, class Map, class Ld, class St>
__device__ __forceinline__ void fft_stage(const FftPlan& P, int s, const Map& M, int lines,
                                          const double2* tw, const Ld& ld, const St& st) {
  constexpr int NB = (kFftPerThread + R - 1) / R;
  const int nr = P.n / R, Ns = P.ns[s], step = nr / Ns, nb = lines * nr;
  const int tid = fresh_tid();
  double2 v[NB][R];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int b = tid + i * NT;
    if (b < nb) {
      int l, j;
      M.split(b, nr, P.m_nr[s], l, j);
#pragma unroll
      for (int q = 0; q < R; ++q) v[i][q] = ld(l, j + q * nr);
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int b = tid + i * NT;
    if (b < nb) {
      int l, j;
      M.split(b, nr, P.m_nr[s], l, j);
      if (Ns > 1) {
        const int t = (j - div_magic(j, P.m_ns[s]) * Ns) * step;
#pragma unroll
        for (int q = 1; q < R; ++q) v[i][q] = cmul(v[i][q], tw[q * t]);
      }
      dft_r(v[i]);
    }
  }
  if (SYNC) __syncthreads();
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int b = tid + i * NT;
    if (b < nb) {
      int l, j;
      M.split(b, nr, P.m_nr[s], l, j);
      const int jd = div_magic(j, P.m_ns[s]), jm = j - jd * Ns;
      const int base = jd * Ns * R + jm;
#pragma unroll
      for (int q = 0; q < R; ++q) st(l, base + q * Ns, v[i][q]);
    }
  }
}

// Which radices a kernel holds: a plan's class (see fft_plan) is 0 for sides
// that are powers of two, 1 with factors 3 and 5, 2 for any other side.
// (One kernel for all took 256 registers, one wavefront per SIMD.)
template <int NT, int CLS, bool SYNC, class Map, class Ld, class St>
__device__ __forceinline__ void fft_stage_any(const FftPlan& P, int s, const Map& M, int lines,
                                              const double2* tw, const Ld& ld, const St& st) {
  const int r = P.radix[s];
  if (r == 8) {
    fft_stage<NT, 8, SYNC>(P, s, M, lines, tw, ld, st);
  } else if (r == 4) {
    fft_stage<NT, 4, SYNC>(P, s, M, lines, tw, ld, st);
  } else if (r == 2) {
    fft_stage<NT, 2, SYNC>(P, s, M, lines, tw, ld, st);
  } else if constexpr (CLS >= 1) {
    if (r == 3)
      fft_stage<NT, 3, SYNC>(P, s, M, lines, tw, ld, st);
    else if (r == 5)
      fft_stage<NT, 5, SYNC>(P, s, M, lines, tw, ld, st);
    else if constexpr (CLS >= 2)
      fft_stage<NT, 7, SYNC>(P, s, M, lines, tw, ld, st);
  }
}

// A stage of any other radix: every output is a direct sum of R terms.
template <int NT, class Map>
__device__ __forceinline__ void fft_stage_sum(const FftPlan& P, int s, const Map& M, int lines,
                                              const double2* tw, double2* buf) {
  const int n = P.n, R = P.radix[s], Ns = P.ns[s], nr = n / R, step = nr / Ns;
  const int tid = fresh_tid();
  double2 out[kFftPerThread];
#pragma unroll
  for (int i = 0; i < kFftPerThread; ++i) {
    const int b = tid + i * NT;
    if (b < lines * n) {
      int l, e;
      M.split(b, n, P.m_n, l, e);
      const int t = div_magic(e, P.m_ns[s]), jm = e - t * Ns;
      const int jd = t / R, k = t - jd * R, j = jd * Ns + jm;
      const int inc = jm * step + k * nr;  // < 2 n
      const int dw = inc >= n ? inc - n : inc;
      double2 acc = make_double2(0.0, 0.0);
      int w = 0;
      for (int q = 0; q < R; ++q) {
        const double2 a = buf[M.at(l, j + q * nr)], c = tw[w];
        acc.x += a.x * c.x - a.y * c.y;
        acc.y += a.x * c.y + a.y * c.x;
        w += dw;
        if (w >= n) w -= n;
      }
      out[i] = acc;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kFftPerThread; ++i) {
    const int b = tid + i * NT;
    if (b < lines * n) {
      int l, e;
      M.split(b, n, P.m_n, l, e);
      buf[M.at(l, e)] = out[i];
    }
  }
  __syncthreads();
}

// Transform `lines` lines: values come from ld(line, element) and end in
// st(line, element, value), or in buf with TO_LDS (a barrier has passed).
// Plans of class 2 with one stage or a direct-sum factor go through LDS at
// both ends.
// All threads call; buf may be written by the next call only after a barrier.
template <int NT, int CLS, bool TO_LDS, class Map, class Ld, class St>
__device__ __forceinline__ void fft_lines(const FftPlan& P, const Map& M, int lines, double2* buf,
                                          const double2* tw, const Ld& ld, const St& st) {
  auto lds_ld = [&](int l, int e) { return buf[M.at(l, e)]; };
  auto lds_st = [&](int l, int e, double2 v) { buf[M.at(l, e)] = v; };
  if (CLS < 2 || (P.nst >= 2 && !P.direct)) {
    fft_stage_any<NT, CLS, false>(P, 0, M, lines, tw, ld, lds_st);
    __syncthreads();
    const int last = TO_LDS ? P.nst : P.nst - 1;
    for (int s = 1; s < last; ++s) {
      fft_stage_any<NT, CLS, true>(P, s, M, lines, tw, lds_ld, lds_st);
      __syncthreads();
    }
    if (!TO_LDS) fft_stage_any<NT, CLS, false>(P, P.nst - 1, M, lines, tw, lds_ld, st);
    return;
  }
  if constexpr (CLS >= 2) {
    const int total = lines * P.n;
    for (int b = fresh_tid(); b < total; b += NT) {
      int l, e;
      M.split(b, P.n, P.m_n, l, e);
      lds_st(l, e, ld(l, e));
    }
    __syncthreads();
    for (int s = 0; s < P.nst; ++s) {
      const int r = P.radix[s];
      if (r <= 5 || r == 7 || r == 8) {
        fft_stage_any<NT, CLS, true>(P, s, M, lines, tw, lds_ld, lds_st);
        __syncthreads();
      } else {
        fft_stage_sum<NT>(P, s, M, lines, tw, buf);
      }
    }
    if (!TO_LDS) {
      for (int b = fresh_tid(); b < total; b += NT) {
        int l, e;
        M.split(b, P.n, P.m_n, l, e);
        st(l, e, lds_ld(l, e));
      }
    }
  }
}

// Launch with `lds` bytes of dynamic LDS (above 64 KB a kernel has to be told).
template <class... KArgs, class... Args>
hipError_t fft_launch(void (*k)(KArgs...), dim3 grid, int nt, size_t lds, hipStream_t s,
                      const Args&... args) {
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, grid, dim3(nt), lds, s, args...);
  return hipGetLastError();
}

// Launch a transform kernel template K<NT, CLS, ...> for a plan: 256 threads
// up to side 256 (four workgroups per CU; 128 threads up to side 128 took 2-15 %
// longer at 96 and 128), 512 above, so that a group of columns stays a whole
// 128-byte line up to side 512.
#define FFT_DISPATCH(P, LAUNCH)                    \
  do {                                             \
    if ((P).nt == 256) {                           \
      if ((P).cls == 0) { LAUNCH(256, 0); }        \
      else if ((P).cls == 1) { LAUNCH(256, 1); }   \
      else { LAUNCH(256, 2); }                     \
    } else {                                       \
      if ((P).cls == 0) { LAUNCH(512, 0); }        \
      else if ((P).cls == 1) { LAUNCH(512, 1); }   \
      else { LAUNCH(512, 2); }                     \
    }                                              \
  } while (0)

// The half spectrum of one field, its planes in up to three pieces of memory.
struct Modes {
  double2 *p0, *p1, *p2;
  int z1, z2;  // planes from z1 on are in p1, from z2 on in p2
  size_t plane;
  __device__ __forceinline__ double2* at(int z) const {
    return z < z1 ? p0 + size_t(z) * plane
                  : (z < z2 ? p1 + size_t(z - z1) * plane : p2 + size_t(z - z2) * plane);
  }
};

__device__ __forceinline__ Modes modes_of(const ModeBuf& B, const FftPlan& P) {
  const int k = B.sc ? B.sc->parity ^ 1 : 0;
  Modes m;
  m.p0 = reinterpret_cast<double2*>(B.seg[k][0]);
  m.p1 = reinterpret_cast<double2*>(B.seg[k][1]);
  m.p2 = reinterpret_cast<double2*>(B.seg[k][2]);
  m.z1 = B.z1;
  m.z2 = B.z2;
  m.plane = size_t(P.n) * P.nhp;
  return m;
}

}  // namespace symlat
