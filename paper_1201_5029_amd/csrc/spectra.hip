// Energy- and number-density spectra of one field (the post-processing
// spectra of Sec. 2.4).  With F_n = DFT(phi_i)/n^3 and P_n = DFT(pi_i)/n^3 of
// the synchronised state, k_eff^2 of the lattice's stencil and m_eff^2 the
// lattice mean of d^2V/dphi_i^2:
//
//   rho_n   = |P_n|^2/(2 a^6) + (k_eff^2/(2 a^2 dx^2) + m_eff^2/2) |F_n|^2
//   omega_n = sqrt(k_eff^2/(a^2 dx^2) + m_eff^2),   n_n = rho_n / omega_n
//
// rho_n is mode n's share of the quadratic energy density (its sum over
// n != 0 is the fluctuations' kinetic, gradient and m_eff^2 energy), n_n the
// corresponding occupation density; both are binned like the field
// spectrum (|n| rounded half away from zero, n = 0 excluded).

#include <algorithm>
#include <cmath>

#include "fft.h"

namespace symlat {

namespace {

// d^2V/dphi_field^2 at fields f; reads only the fields it depends on (see
// d2v_reads).
template <int KIND, int NF, typename T>
__device__ __forceinline__ T d2v_one(const T (&f)[NF], const PotT<T>& P, int field) {
  if constexpr (KIND == SL_POT_FREE) {
    return P.p[field];
  } else if constexpr (KIND == SL_POT_CHAOTIC2) {
    return field == 0 ? P.p[0] + P.p[1] * f[1] * f[1] : P.p[1] * f[0] * f[0];
  } else if constexpr (KIND == SL_POT_OSCILLON) {
    const T x2 = f[0] * f[0];
    return P.p[0] - T(3) * P.p[1] * x2 + T(5) * P.p[2] * x2 * x2;
  } else {
    const T m2 = P.p[0], K = P.p[1], invM2 = P.p[2];
    const T u = T(0.5) * (f[0] * f[0] + f[1] * f[1]);
    if (!(u > T(0))) return T(0);
    const T g = field == 0 ? f[0] : f[1];
    return m2 * (T(1) + K + K * dev_log<T>(u * invM2)) + m2 * K * g * g / u;
  }
}

// Whether d^2V/dphi_field^2 depends on field i.
template <int KIND>
__device__ __forceinline__ bool d2v_reads(int field, int i) {
  if constexpr (KIND == SL_POT_FREE) return false;
  if constexpr (KIND == SL_POT_CHAOTIC2) return i != field;
  return true;
}

struct Bufs4 {
  const void* phi[2];
  const void* pi[2];
};

// Per-block compensated sums of d^2V/dphi_field^2 at the synchronised fields.
// A block takes whole chunks of planes (no division per site); it reads only
// the fields the derivative depends on: one of two for the chaotic model,
// none for free fields.  256^3 FP64, chaotic model: 67 us, 4 TB/s (173 us with
// both fields, one block per CU and a 64-bit division per site).
template <typename T, int NF, int KIND>
__global__ __launch_bounds__(kBlock) void meff_kernel(Bufs4 B, const DevScalars* sc, PotArgs prm,
                                                     int field, int n, int zs, int chunks,
                                                     double* part) {
  __shared__ KSum scratch[4];
  const int par = sc->parity;
  const T* phi = static_cast<const T*>(B.phi[par]);
  const T* pi = static_cast<const T*>(B.pi[par]);
  const double c = sc->c_pend;
  PotT<double> pot;
#pragma unroll
  for (int i = 0; i < kMaxFields; ++i) pot.p[i] = prm.p[i];
  double off[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) off[i] = sc->off_phi[i] + c * sc->off_pi[i];
  const size_t n2 = size_t(n) * n;
  const size_t per = (n2 + chunks - 1) / chunks;
  KSum acc[1] = {{0.0, 0.0}};
  for (int w = int(blockIdx.x); w < n * chunks; w += int(gridDim.x)) {
    const int z = w / chunks;
    const size_t r0 = size_t(w - z * chunks) * per, r1 = r0 + per < n2 ? r0 + per : n2;
#pragma unroll 4
    for (size_t r = r0 + threadIdx.x; r < r1; r += kBlock) {
      double f[NF];
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        f[i] = 0.0;
        if (d2v_reads<KIND>(field, i)) {
          const size_t o = (size_t(z) * zs + i) * n2 + r;
          f[i] = off[i] + fma(c, double(pi[o]), double(phi[o]));
        }
      }
      kadd(acc[0], d2v_one<KIND, NF, double>(f, pot, field));
    }
  }
  block_reduce<1>(acc, scratch);
  if (threadIdx.x == 0) {
    part[2 * size_t(blockIdx.x)] = acc[0].s;
    part[2 * size_t(blockIdx.x) + 1] = acc[0].c;
  }
}

__global__ __launch_bounds__(kBlock) void meff_finalize_kernel(const double* part, int nblocks,
                                                              double inv_n3, double* m2) {
  __shared__ KSum scratch[4];
  KSum v[1] = {{0.0, 0.0}};
  for (int b = int(threadIdx.x); b < nblocks; b += kBlock)
    v[0] = kcombine(v[0], KSum{part[2 * size_t(b)], part[2 * size_t(b) + 1]});
  block_reduce<1>(v, scratch);
  if (threadIdx.x == 0) *m2 = (v[0].s + v[0].c) * inv_n3;
}

// Shell index of |n|^2 = m: round(|n|) half away from zero, in integers
// (m < 2^20: the float root is within one of the integer one).
__device__ __forceinline__ int shell_of(int m) {
  int b = int(sqrtf(float(m)));
  if (b * b > m) --b;
  if ((b + 1) * (b + 1) <= m) ++b;
  return m > b * b + b ? b + 1 : b;
}

// What a bin sums, by kind: the field spectrum alone; the field's part of the
// three spectra; the momentum's part of the energy and number spectra (both
// are linear in |F|^2 and |P|^2, so field and momentum are transformed one
// after the other in the same memory).
enum { kBinField = 0, kBinSpectraField = 1, kBinSpectraMomentum = 2 };
constexpr int bin_values(int kind) { return kind == kBinField ? 3 : (kind == kBinSpectraField ? 5 : 2); }

struct BinArgs {
  int nbe;           // bins that can hold a mode and are asked for
  int stencil_kind;
  double stc[4];
  double inv_n6, inv_dx2;
  const DevScalars* sc;
  const double* m2;  // m_eff^2
};

// |n| and the mode counts of the bins depend on n alone: 1/48 of the modes,
// the folded wave numbers a >= b >= c of min(n_d, n - n_d), stand for all
// (their permutations, and two signs for each value but 0 and n/2).  A thread
// takes 16 values of c; 8.4 M modes at 256^3 would be two atomics each.
template <int NT>
__device__ void count_modes(int n, int nbe, double* ksum, double* count) {
  const int h = n / 2, cc = h / 16 + 1, total = (h + 1) * (h + 1) * cc;
  for (int t = int(blockIdx.x) * NT + int(threadIdx.x); t < total; t += int(gridDim.x) * NT) {
    const int a = t / ((h + 1) * cc), r = t - a * (h + 1) * cc, b = r / cc, c0 = (r - b * cc) * 16;
    if (b > a) continue;
    const int mab = a * a + b * b, sab = (a == 0 || 2 * a == n ? 1 : 2) * (b == 0 || 2 * b == n ? 1 : 2);
    for (int c = c0; c < c0 + 16 && c <= b; ++c) {
      const int m = mab + c * c;
      if (m == 0) continue;
      const int bin = shell_of(m);
      if (bin >= nbe) continue;
      const int perms = a == b ? (b == c ? 1 : 3) : (b == c ? 3 : 6);
      const double w = double(perms * sab * (c == 0 || 2 * c == n ? 1 : 2));
      unsafeAtomicAdd(&ksum[bin], w * sqrt(double(m)));
      unsafeAtomicAdd(&count[bin], w);
    }
  }
}

// z pass of the forward transform with the binning as its output: the modes
// leave the last stage in registers and are added to the workgroup's bins in
// LDS (hardware FP64 atomics), so they are never written back.  A mode with
// 0 < kx < n/2 stands for two (its conjugate has the same |F|, |n| and
// k_eff^2).  Each workgroup writes one row of partial bins; as many
// workgroups as are resident, so that the rows stay few.  It is bound by the
// energy of each mode (a root and a reciprocal) and the atomics: 83 us for a
// field and 67 us for its momentum at 256^3, against 50 us for the same pass
// with nothing but the transform; a complex z pass of each and a binning pass
// over both took 2 x 266 + 391 us.
template <int NT, int CLS, int KIND>
__global__ __launch_bounds__(NT, NT == 512 ? 4 : 3) void bin_columns_kernel(FftPlan P, ModeBuf B,
                                                         const double2* __restrict__ twg,
                                                         const double* __restrict__ axg, int lg,
                                                         BinArgs A) {
  extern __shared__ double2 smem[];
  constexpr int NV = bin_values(KIND);
  const int n = P.n, L = 1 << lg, total = n * P.nhp, nbe = A.nbe;
  double2* tw = smem;
  double2* buf = smem + n;
  const int vals = L * n;
  double* ax = reinterpret_cast<double*>(buf + vals + (vals >> 3));
  double* bins = ax + n;
  for (int i = int(threadIdx.x); i < n; i += NT) {
    tw[i] = twg[i];
    ax[i] = axg[i];
  }
  for (int i = int(threadIdx.x); i < NV * nbe; i += NT) bins[i] = 0.0;
  const Modes m = modes_of(B, P);
  const ColMap M{lg};
  // coefficients of the energy of a mode: rho = cp |P|^2 + (ck k2 + cm) |F|^2,
  // omega^2 = wk k2 + m2
  double cp = 0.0, ck = 0.0, cm = 0.0, wk = 0.0, m2 = 0.0;
  if constexpr (KIND != kBinField) {
    const double a = A.sc->a, a2 = a * a;
    m2 = *A.m2;
    cp = 1.0 / (2.0 * a2 * a2 * a2);
    ck = A.inv_dx2 / (2.0 * a2);
    cm = 0.5 * m2;
    wk = A.inv_dx2 / a2;
  }
  __syncthreads();
  if constexpr (KIND != kBinSpectraMomentum)
    count_modes<NT>(n, nbe, bins + (NV - 2) * nbe, bins + (NV - 1) * nbe);
  for (int g0 = int(blockIdx.x) * L; g0 < total; g0 += int(gridDim.x) * L) {
    const int id = g0 + (int(threadIdx.x) & (L - 1));
    const int idc = id < total ? id : total - 1;
    const int uy = div_magic(idc, P.m_nhp), ux = idc - uy * P.nhp;
    const bool own = id < total && ux < P.nh;
    const int ky = 2 * uy >= n ? uy - n : uy;
    const int mxy = ux * ux + ky * ky;
    const double w = (ux == 0 || 2 * ux == n) ? 1.0 : 2.0;
    const double axx = ax[own ? ux : 0], axy = ax[uy];
    auto ld = [&](int, int e) { return m.at(e)[idc]; };
    auto st = [&](int, int uz, double2 v) {
      const int kz = 2 * uz >= n ? uz - n : uz;
      const int mm = mxy + kz * kz;
      if (!own || mm == 0) return;
      const int b = shell_of(mm);
      if (b >= nbe) return;
      const double f2 = w * (v.x * v.x + v.y * v.y) * A.inv_n6;
      if constexpr (KIND == kBinField) {
        unsafeAtomicAdd(&bins[b], f2);
      } else {
        double k2;
        if (A.stencil_kind == 0) {
          k2 = ax[uz] + axy + axx;
        } else {
          const double cz = ax[uz];
          k2 = -(A.stc[0] + 2.0 * A.stc[1] * (cz + axy + axx) +
                 4.0 * A.stc[2] * (cz * axy + cz * axx + axy * axx) + 8.0 * A.stc[3] * cz * axy * axx);
        }
        const double w2 = fma(wk, k2, m2);
        const double rho = KIND == kBinSpectraField ? fma(ck, k2, cm) * f2 : cp * f2;
        const double num = w2 > 0.0 ? rho * rsqrt(w2) : 0.0;
        int at = b;
        if constexpr (KIND == kBinSpectraField) {
          unsafeAtomicAdd(&bins[at], f2);
          at += nbe;
        }
        unsafeAtomicAdd(&bins[at], rho);
        unsafeAtomicAdd(&bins[at + nbe], num);
      }
    };
    fft_lines<NT, CLS, false>(P, M, L, buf, tw, ld, st);
    __syncthreads();
  }
  const int k = B.sc ? B.sc->parity ^ 1 : 0;
  double* out = B.part[k] + size_t(blockIdx.x) * NV * nbe;
  for (int i = int(threadIdx.x); i < NV * nbe; i += NT) out[i] = bins[i];
}

// Sum the rows of partial bins: kFinBins bins per workgroup, 256 threads striding
// through the rows of each (17 us for 768 rows of 5 + 2 sums, 222 bins; 38 us
// with 16 bins to a workgroup, where 14 CUs worked; one thread per bin took 100
// us for 256 rows of 5); out =
// [k | <|F|^2> (| <rho> | <n>) | count], nbe values each, then m_eff^2 (NV = 5)
// and the scalars.  rows2 > 0: rows of the momentum's part follow.
constexpr int kFinBins = 4;
template <int NV>
__global__ __launch_bounds__(1024) void bin_finalize_kernel(ModeBuf B, int rows, int rows2, int nbe,
                                                            double L, const DevScalars* sc,
                                                            const double* m2, double* out) {
  __shared__ KSum sh[NV][16][kFinBins];
  constexpr int G = 1024 / kFinBins;
  const int t = int(threadIdx.x), i = t % kFinBins, g = t / kFinBins, wave = t >> 6;
  const int b = int(blockIdx.x) * kFinBins + i;
  const bool own = b < nbe;
  const double* p1 = B.part[B.sc ? B.sc->parity ^ 1 : 0] + b;
  const double* p2 = p1 + size_t(rows) * NV * nbe;
  if (blockIdx.x == 0) {
    double* tail = out + size_t(NV) * nbe;
    if (NV == 5 && t == 64) tail[0] = *m2;
    const int w = t - 128;
    if (w >= 0 && w < int(sizeof(DevScalars) / sizeof(uint64_t)))
      reinterpret_cast<uint64_t*>(tail + (NV == 5 ? 1 : 0))[w] = reinterpret_cast<const uint64_t*>(sc)[w];
  }
  KSum v[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = KSum{0.0, 0.0};
  if (own) {
#pragma unroll 4
    for (int r = g; r < rows; r += G) {
#pragma unroll
      for (int q = 0; q < NV; ++q) kadd(v[q], p1[(size_t(r) * NV + q) * nbe]);
    }
    if constexpr (NV == 5) {
#pragma unroll 4
      for (int r = g; r < rows2; r += G) {
        kadd(v[1], p2[size_t(r) * 2 * nbe]);
        kadd(v[2], p2[(size_t(r) * 2 + 1) * nbe]);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < NV; ++q) {
#pragma unroll
    for (int o = kFinBins; o <= 32; o <<= 1) {  // the row groups of a wavefront
      KSum w;
      w.s = __shfl_xor(v[q].s, o, 64);
      w.c = __shfl_xor(v[q].c, o, 64);
      v[q] = kcombine(v[q], w);
    }
    if ((t & 63) < kFinBins) sh[q][wave][i] = v[q];
  }
  __syncthreads();
  if (t >= kFinBins || !own) return;
  double tot[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    KSum s = sh[q][0][i];
#pragma unroll
    for (int k = 1; k < 16; ++k) s = kcombine(s, sh[q][k][i]);
    tot[q] = s.s + s.c;
  }
  // sums: |F|^2 (rho, n), |n|, count
  const double cnt = tot[NV - 1], inv = cnt > 0 ? 1.0 / cnt : 0.0;
  out[b] = 2.0 * M_PI * tot[NV - 2] * inv / L;
#pragma unroll
  for (int q = 0; q < NV - 2; ++q) out[(q + 1) * nbe + b] = tot[q] * inv;
  out[(NV - 1) * nbe + b] = cnt;
}

template <typename T, int NF, int KIND>
hipError_t meff_t(const LatView& v, int field, double* part, double* m2, hipStream_t s) {
  const double n3 = double(v.n) * v.n * v.n;
  const size_t n2 = size_t(v.n) * v.n;
  Bufs4 B;
  for (int k = 0; k < 2; ++k) {
    B.phi[k] = v.phi[k];
    B.pi[k] = v.pi[k];
  }
  // chunks of at least 1024 sites, about two per block at most
  int chunks = int(std::min<size_t>((n2 + 1023) / 1024, size_t(2 * kMeffBlocks / v.n)));
  if (chunks < 1) chunks = 1;
  const int nb = v.n * chunks < kMeffBlocks ? v.n * chunks : kMeffBlocks;
  hipLaunchKernelGGL((meff_kernel<T, NF, KIND>), dim3(nb), dim3(kBlock), 0, s, B, v.sc, v.prm, field, v.n,
                     v.zs, chunks, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(meff_finalize_kernel, dim3(1), dim3(kBlock), 0, s, part, nb, 1.0 / n3, m2);
  return hipGetLastError();
}

template <typename T>
hipError_t meff_prec(const LatView& v, int field, double* part, double* m2, hipStream_t s) {
  switch (v.pot) {
    case SL_POT_CHAOTIC2: return meff_t<T, 2, SL_POT_CHAOTIC2>(v, field, part, m2, s);
    case SL_POT_OSCILLON: return meff_t<T, 1, SL_POT_OSCILLON>(v, field, part, m2, s);
    case SL_POT_QBALL_LOG: return meff_t<T, 2, SL_POT_QBALL_LOG>(v, field, part, m2, s);
    default: return meff_t<T, 1, SL_POT_FREE>(v, field, part, m2, s);  // reads no field
  }
}

template <int KIND>
hipError_t bin_columns(const FftPlan& P, const ModeBuf& B, const double2* tw, const double* ax, int rows,
                       const BinArgs& A, hipStream_t s) {
  const int lg = fft_column_lines_log2(P);
  const size_t lds = fft_lds_bytes(P.n, 1 << lg) +
                     (size_t(P.n) + size_t(bin_values(KIND)) * A.nbe) * sizeof(double);
#define BIN_LAUNCH(NT, CLS) return fft_launch(bin_columns_kernel<NT, CLS, KIND>, dim3(rows), NT, lds, s, P, B, tw, ax, lg, A)
  FFT_DISPATCH(P, BIN_LAUNCH);
#undef BIN_LAUNCH
}

BinArgs bin_args(const LatView& v, int nbe, const double* m2) {
  BinArgs A;
  const double n3 = double(v.n) * v.n * v.n;
  A.nbe = nbe;
  A.stencil_kind = v.st.kind;
  for (int k = 0; k < 4; ++k) A.stc[k] = v.st.c[k];
  A.inv_n6 = 1.0 / (n3 * n3);
  A.inv_dx2 = v.bg.inv_dx2;
  A.sc = v.sc;
  A.m2 = m2;
  return A;
}

}  // namespace

int spectrum_bins(int n, int nbins) {
  const int most = int(std::sqrt(3.0) * (n / 2)) + 2;  // one past the corner mode's bin
  return nbins < most ? nbins : most;
}

int bin_rows_max(const FftPlan& P) {
  // three workgroups of 256 threads or two of 512 per CU.  With five values of
  // all bins the LDS of sides from about 400 up leaves room for one, and the
  // 512 run in two rounds: 256 rows took the same time at 512^3 (3435 us) and
  // longer at 448^3 (2414 against 2292) and 640^3 (8157 and 7485), where the
  // momentum's pass has room for two.
  const int lg = fft_column_lines_log2(P), groups = (P.n * P.nhp + (1 << lg) - 1) >> lg;
  const int most = P.nt == 256 ? 768 : 512;
  return groups < most ? groups : most;
}

hipError_t launch_meff(const LatView& v, int field, double* part, double* m2_dev, hipStream_t s) {
  return v.prec == SL_FP32 ? meff_prec<float>(v, field, part, m2_dev, s)
                           : meff_prec<double>(v, field, part, m2_dev, s);
}

hipError_t launch_spectrum_bins(const LatView& v, const FftPlan& P, const ModeBuf& B, const double2* tw,
                                const double* ax, int nbe, int rows, double* out3, hipStream_t s) {
  const hipError_t e = bin_columns<kBinField>(P, B, tw, ax, rows, bin_args(v, nbe, nullptr), s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(bin_finalize_kernel<3>, dim3((nbe + kFinBins - 1) / kFinBins), dim3(1024), 0, s, B, rows, 0, nbe, v.bg.L,
                     v.sc, static_cast<const double*>(nullptr), out3);
  return hipGetLastError();
}

hipError_t launch_mode_bins(const LatView& v, int momentum, const FftPlan& P, const ModeBuf& B,
                            const double2* tw, const double* ax, int nbe, int rows, const double* m2_dev,
                            hipStream_t s) {
  if (!momentum) return bin_columns<kBinSpectraField>(P, B, tw, ax, rows, bin_args(v, nbe, m2_dev), s);
  ModeBuf after = B;  // the momentum's rows follow the field's
  for (int k = 0; k < 2; ++k) after.part[k] = B.part[k] + size_t(rows) * 5 * nbe;
  return bin_columns<kBinSpectraMomentum>(P, after, tw, ax, rows, bin_args(v, nbe, m2_dev), s);
}

hipError_t launch_mode_bins_finalize(const LatView& v, const ModeBuf& B, int nbe, int rows,
                                     const double* m2_dev, double* out5,
                                     hipStream_t s) {
  hipLaunchKernelGGL(bin_finalize_kernel<5>, dim3((nbe + kFinBins - 1) / kFinBins), dim3(1024), 0, s, B, rows, rows, nbe, v.bg.L,
                     v.sc, m2_dev, out5);
  return hipGetLastError();
}

}  // namespace symlat
