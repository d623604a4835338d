// Initial state on the device.
//
// Random numbers: counter-based SplitMix64 (Steele, Lea & Flood, OOPSLA 2014:
// the k-th output from a seed is the published finaliser applied to
// seed + k * 0x9E3779B97F4A7C15) with 53-bit uniforms in (0, 1] and
// Box-Muller normals.  Draw r (0/1) of component c (0/1) for field i at
// linear index idx of an N-entry array uses output number
// 4 (i N + idx) + 2c + r + 1, so results do not depend on the launch shape.
//
// The vacuum modes are drawn where the inverse transform's first pass would
// read them (see fft.h): no mode array is written before it.

#include "fft.h"

namespace symlat {

namespace {

__device__ __forceinline__ uint64_t splitmix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ double uniform01(uint64_t seed, uint64_t counter) {
  const uint64_t x = splitmix64(seed + (counter + 1ull) * 0x9E3779B97F4A7C15ull);
  return (double((x >> 11)) + 1.0) * 0x1.0p-53;
}

// A normal times sqrt(var): the variance goes under Box-Muller's root.
__device__ __forceinline__ double normal(uint64_t seed, uint64_t field, uint64_t count,
                                         uint64_t idx, uint64_t comp, double var) {
  const uint64_t base = 4ull * (field * count + idx) + 2ull * comp;
  const double u1 = uniform01(seed, base);
  const double u2 = uniform01(seed, base + 1ull);
  return sqrt(-2.0 * var * log(u1)) * cospi(2.0 * u2);
}

template <typename T>
__global__ void fill_homogeneous_kernel(void* phi0, void* pi0, int nf, int zs, size_t n2,
                                        size_t n3, PotArgs v0, PotArgs p0, Offsets off) {
  T* phi = static_cast<T*>(phi0);
  T* pi = static_cast<T*>(pi0);
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n3 * nf; e += stride) {
    const int i = int(e / n3);  // field i, site e - i n^3
    const size_t d = field_site(i, e - size_t(i) * n3, zs, n2);
    phi[d] = static_cast<T>(v0.p[i] - off.phi[i]);
    pi[d] = static_cast<T>(p0.p[i] - off.pi[i]);
  }
}

struct VacArgs {
  double m2eff, half_amp2, inv_dx2;  // half_amp2 = A^2/(2 L^3)
  uint64_t seed;
  int field, stencil_kind;
  double stc[4];
};

// f_n for the modes of one field with kx = 0 .. n/2, and their inverse
// z pass: E|f_n|^2 = A^2/(2 omega_n L^3), omega_n^2 = k_eff^2/dx^2 + m_eff^2,
// f_0 = 0, f_{-n} = conj(f_n), real on self-conjugate modes; each +-n pair
// draws at its smaller linear index, so the conjugate half that the planes
// kx = 0 and n/2 hold comes out the same.  k_eff^2 is minus the eigenvalue of
// the lattice Laplacian on the mode: for the 7-point stencil sum_d 4 sin^2(pi
// n_d/N), for a general member of the cubic family -(c0 + 2 c1 sum cos + 4 c2
// sum cos cos + 8 c3 prod cos).  Bound by the draws (two roots, logarithms
// and cosines and four 64-bit mixers a mode): 41 us a field at 128^3, and the
// y and x passes 12 + 15 us; drawing all n^3 modes took 57 us, the complex
// axis passes 3 x 27 us and storing the field 8 us.
template <int NT, int CLS>
__global__ __launch_bounds__(NT, NT == 512 ? 4 : 3) void vacuum_columns_kernel(
    FftPlan P, ModeBuf B, const double2* __restrict__ twg, const double* __restrict__ ax, int lg,
    VacArgs A) {
  extern __shared__ double2 smem[];
  const int n = P.n, L = 1 << lg, total = n * P.nhp;
  double2* tw = smem;
  double2* buf = smem + n;
  for (int i = int(threadIdx.x); i < n; i += NT) tw[i] = twg[i];
  const Modes m = modes_of(B, P);
  const ColMap M{lg};
  const uint64_t n3 = uint64_t(n) * n * n;
  __syncthreads();
  for (int g0 = int(blockIdx.x) * L; g0 < total; g0 += int(gridDim.x) * L) {
    const int id = g0 + (int(threadIdx.x) & (L - 1));
    const int idc = id < total ? id : total - 1;
    const int uy = div_magic(idc, P.m_nhp), ux = idc - uy * P.nhp;
    const bool own = id < total && ux < P.nh;
    const double axx = ax[own ? ux : 0], axy = ax[uy];
    const int mx = ux ? n - ux : 0, my = uy ? n - uy : 0;
    auto ld = [&](int, int uz) {
      if (!own) return make_double2(0.0, 0.0);
      const int mz = uz ? n - uz : 0;
      const unsigned e = (unsigned(uz) * n + uy) * n + ux, neg = (unsigned(mz) * n + my) * n + mx;
      const unsigned canon = e < neg ? e : neg;
      const double az = ax[uz];
      const double keff2 =
          A.stencil_kind == 0
              ? az + axy + axx
              : -(A.stc[0] + 2.0 * A.stc[1] * (az + axy + axx) +
                  4.0 * A.stc[2] * (az * axy + az * axx + axy * axx) + 8.0 * A.stc[3] * az * axy * axx);
      const double w2 = fma(keff2, A.inv_dx2, A.m2eff);
      // E|f|^2, split evenly over two parts unless the mode is real
      double var = w2 > 0.0 && e != 0 ? A.half_amp2 * rsqrt(w2) : 0.0;
      if (neg != e) var *= 0.5;
      const double re = normal(A.seed, uint64_t(A.field), n3, canon, 0, var);
      if (neg == e) return make_double2(0.0, re);
      const double im = normal(A.seed, uint64_t(A.field), n3, canon, 1, var);
      // real and imaginary parts exchanged: the forward stages invert
      return make_double2(e == canon ? im : -im, re);
    };
    auto st = [&](int, int uz, double2 v) {
      if (own) m.at(uz)[idc] = make_double2(v.y, v.x);
    };
    fft_lines<NT, CLS, false>(P, M, L, buf, tw, ld, st);
    __syncthreads();
  }
}

__global__ __launch_bounds__(kBlock) void white_kernel(double* g, size_t n3, int field,
                                                      uint64_t seed, double* partials) {
  __shared__ KSum scratch[4];
  KSum acc[1] = {{0.0, 0.0}};
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n3; e += stride) {
    const double v = normal(seed, uint64_t(field), n3, e, 0, 1.0);
    g[e] = v;
    kadd(acc[0], v);
  }
  block_reduce<1>(acc, scratch);
  if (threadIdx.x == 0) {
    partials[2 * blockIdx.x] = acc[0].s;
    partials[2 * blockIdx.x + 1] = acc[0].c;
  }
}

__global__ __launch_bounds__(kBlock) void mean_finalize_kernel(const double* partials, int nblocks,
                                                              double inv_count, double* mean) {
  __shared__ KSum scratch[4];
  KSum v[1] = {{0.0, 0.0}};
  for (int b = threadIdx.x; b < nblocks; b += kBlock)
    v[0] = kcombine(v[0], KSum{partials[2 * b], partials[2 * b + 1]});
  block_reduce<1>(v, scratch);
  if (threadIdx.x == 0) *mean = (v[0].s + v[0].c) * inv_count;
}

template <typename T>
__global__ void white_store_kernel(void* phi0, const double* g, const double* mean, size_t n3,
                                   size_t n2, int zs, int field, double base, double amp) {
  T* phi = static_cast<T*>(phi0);
  const double mu = *mean;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n3; e += stride)
    phi[field_site(field, e, zs, n2)] = static_cast<T>(base + amp * (g[e] - mu));
}

int grid_for(size_t count) {
  size_t nb = (count + kBlock - 1) / kBlock;
  if (nb > 4096) nb = 4096;
  if (nb < 1) nb = 1;
  return int(nb);
}

}  // namespace

hipError_t launch_fill_homogeneous(const LatView& v, const double* phi0, const double* pi0,
                                   const Offsets& off, hipStream_t s) {
  PotArgs a{}, b{};
  for (int i = 0; i < v.nf; ++i) {
    a.p[i] = phi0[i];
    b.p[i] = pi0[i];
  }
  const size_t n3 = size_t(v.n) * v.n * v.n;
  const int nb = grid_for(n3 * v.nf);
  if (v.prec == SL_FP32)
    hipLaunchKernelGGL(fill_homogeneous_kernel<float>, dim3(nb), dim3(kBlock), 0, s, v.phi[0],
                       v.pi[0], v.nf, v.zs, size_t(v.n) * v.n, n3, a, b, off);
  else
    hipLaunchKernelGGL(fill_homogeneous_kernel<double>, dim3(nb), dim3(kBlock), 0, s, v.phi[0],
                       v.pi[0], v.nf, v.zs, size_t(v.n) * v.n, n3, a, b, off);
  return hipGetLastError();
}

hipError_t launch_vacuum_columns(const LatView& v, int field, double m2eff, double amp, uint64_t seed,
                                 const FftPlan& P, const ModeBuf& B, const double2* tw,
                                 const double* ax, hipStream_t s) {
  VacArgs A;
  A.m2eff = m2eff;
  // in extended precision: L^3 alone leaves the range of doubles for sides whose
  // modes are ordinary numbers
  const long double L1 = v.bg.L;
  A.half_amp2 = double(0.5L * amp * amp / (L1 * L1 * L1));
  A.inv_dx2 = v.bg.inv_dx2;
  A.seed = seed;
  A.field = field;
  A.stencil_kind = v.st.kind;
  for (int k = 0; k < 4; ++k) A.stc[k] = v.st.c[k];
  const int lg = fft_column_lines_log2(P), L = 1 << lg, groups = (P.n * P.nhp + L - 1) / L;
  const dim3 grid(groups < kFftGridMax ? groups : kFftGridMax);
  const size_t lds = fft_lds_bytes(P.n, L);
#define VAC_LAUNCH(NT, CLS) return fft_launch(vacuum_columns_kernel<NT, CLS>, grid, NT, lds, s, P, B, tw, ax, lg, A)
  FFT_DISPATCH(P, VAC_LAUNCH);
#undef VAC_LAUNCH
}

hipError_t launch_white(const LatView& v, double* gbuf, double* mean_dev, int field, double base,
                        double amp, uint64_t seed, hipStream_t s) {
  const size_t n3 = size_t(v.n) * v.n * v.n;
  const int nb = grid_for(n3) > 1024 ? 1024 : grid_for(n3);
  hipLaunchKernelGGL(white_kernel, dim3(nb), dim3(kBlock), 0, s, gbuf, n3, field, seed,
                     v.partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(mean_finalize_kernel, dim3(1), dim3(kBlock), 0, s, v.partials, nb,
                     1.0 / double(n3), mean_dev);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (v.prec == SL_FP32)
    hipLaunchKernelGGL(white_store_kernel<float>, dim3(grid_for(n3)), dim3(kBlock), 0, s,
                       v.phi[0], gbuf, mean_dev, n3, size_t(v.n) * v.n, v.zs, field, base, amp);
  else
    hipLaunchKernelGGL(white_store_kernel<double>, dim3(grid_for(n3)), dim3(kBlock), 0, s,
                       v.phi[0], gbuf, mean_dev, n3, size_t(v.n) * v.n, v.zs, field, base, amp);
  return hipGetLastError();
}

}  // namespace symlat
