// Axis passes of the half-spectrum transforms (see fft.h) and the host side of
// their plans.

#include "fft.h"

namespace symlat {

namespace {

__global__ void fft_tables_kernel(int n, Stencil st, double2* tw, double* ax) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m < n) {
    const double t = 2.0 * double(m) / n;
    tw[m] = make_double2(cospi(t), -sinpi(t));
    const double s = sinpi(double(m) / n);
    ax[m] = st.kind == 0 ? 4.0 * s * s : cospi(t);
  }
}

// Rows of one field of a lattice at the synchronised state, less the value at
// site 0 (a constant moves only the k = 0 mode, which no caller uses, and the
// rounding of the transform is relative to the largest value): phi + c pi, or
// the stored momenta.  (Which of them is a template parameter: a branch around
// the field's load made each value wait for its own.)
template <typename T, bool MOMENTUM>
struct LatticeRows {
  const void* phi[2];
  const void* pi[2];
  const DevScalars* sc;
  int zs, field;
  struct View {
    const T *f, *p;
    double c, shift;
    size_t n, n2, zs;
    __device__ __forceinline__ double raw(size_t o) const {
      const double q = double(p[o]);
      if constexpr (MOMENTUM) return q;
      return fma(c, q, double(f[o]));
    }
    __device__ __forceinline__ double operator()(int z, int y, int x) const {
      return raw(size_t(z) * zs * n2 + size_t(y) * n + x) - shift;
    }
  };
  __device__ View view(int n) const {
    View v;
    const int par = sc->parity;
    v.n = n;
    v.n2 = size_t(n) * n;
    v.zs = zs;
    v.f = static_cast<const T*>(phi[par]) + size_t(field) * v.n2;
    v.p = static_cast<const T*>(pi[par]) + size_t(field) * v.n2;
    v.c = sc->c_pend;
    v.shift = v.raw(0);
    return v;
  }
};

// Rows of a plain real array [z][y][x] less a value in device memory.
struct ArrayRows {
  const double* r;
  const double* shift;
  struct View {
    const double* r;
    double shift;
    size_t n;
    __device__ __forceinline__ double operator()(int z, int y, int x) const {
      return r[(size_t(z) * n + y) * n + x] - shift;
    }
  };
  __device__ View view(int n) const { return View{r, *shift, size_t(n)}; }
};

// Forward x pass: pairs of real rows of `src` into half-spectrum rows.
template <int NT, int CLS, class Src>
__global__ __launch_bounds__(NT, NT == 512 ? 4 : 3) void r2c_rows_kernel(FftPlan P, Src src, ModeBuf B,
                                                      const double2* __restrict__ twg, int lines,
                                                      int npairs) {
  extern __shared__ double2 smem[];
  const int n = P.n, nh = P.nh, hy = (n + 1) / 2;
  double2* tw = smem;
  double2* buf = smem + n;
  for (int i = int(threadIdx.x); i < n; i += NT) tw[i] = twg[i];
  const auto S = src.view(n);
  const Modes out = modes_of(B, P);
  const RowMap M{n};
  __syncthreads();
  for (int g0 = int(blockIdx.x) * lines; g0 < npairs; g0 += int(gridDim.x) * lines) {
    const int cnt = min(lines, npairs - g0);
    auto ld = [&](int l, int e) {
      const int z = div_magic(g0 + l, P.m_hy), y = 2 * (g0 + l - z * hy);
      const bool two = y + 1 < n;  // else the row again (no branch around a load)
      const double a = S(z, y, e), b = S(z, two ? y + 1 : y, e);
      return make_double2(a, two ? b : 0.0);
    };
    auto none = [](int, int, double2) {};
    fft_lines<NT, CLS, true>(P, M, cnt, buf, tw, ld, none);
    for (int b = fresh_tid(); b < cnt * nh; b += NT) {
      const int l = div_magic(b, P.m_nh), k = b - l * nh;
      const double2 a = buf[M.at(l, k)], c = buf[M.at(l, k ? n - k : 0)];
      const int z = div_magic(g0 + l, P.m_hy), y = 2 * (g0 + l - z * hy);
      double2* row = out.at(z) + size_t(y) * P.nhp + k;
      row[0] = make_double2(0.5 * (a.x + c.x), 0.5 * (a.y - c.y));
      if (y + 1 < n) row[P.nhp] = make_double2(0.5 * (a.y + c.y), 0.5 * (c.x - a.x));
    }
    __syncthreads();
  }
}

// Field i of a lattice's buffer 0 as the target of an inverse transform.
template <typename T>
struct LatticeSink {
  void* phi;
  void* pi;
  int zs, field;
  double base, pi_value;
  __device__ __forceinline__ void put(int n, int z, int y, int x, double v) const {
    const size_t o = ((size_t(z) * zs + field) * n + y) * n + x;
    static_cast<T*>(phi)[o] = static_cast<T>(base + v);
    static_cast<T*>(pi)[o] = static_cast<T>(pi_value);
  }
};

// A plain real array [z][y][x] = scale * transform + *add (device memory).
struct ArraySink {
  double* r;
  double scale;
  const double* add;
  __device__ __forceinline__ void put(int n, int z, int y, int x, double v) const {
    r[(size_t(z) * n + y) * n + x] = fma(v, scale, *add);
  }
};

// Inverse x pass: half-spectrum rows A, B of two neighbouring rows as the
// complex row A + i B, whose inverse transform holds one row in its real and
// the other in its imaginary part.  Z_k for k > n/2 is conj(A_{n-k}) +
// i conj(B_{n-k}).  Real and imaginary parts exchanged, as in the columns.
template <int NT, int CLS, class Sink>
__global__ __launch_bounds__(NT, NT == 512 ? 4 : 3) void c2r_rows_kernel(FftPlan P, ModeBuf B, Sink sink,
                                                      const double2* __restrict__ twg, int lines,
                                                      int npairs) {
  extern __shared__ double2 smem[];
  const int n = P.n, hy = (n + 1) / 2;
  double2* tw = smem;
  double2* buf = smem + n;
  for (int i = int(threadIdx.x); i < n; i += NT) tw[i] = twg[i];
  const Modes in = modes_of(B, P);
  const RowMap M{n};
  __syncthreads();
  for (int g0 = int(blockIdx.x) * lines; g0 < npairs; g0 += int(gridDim.x) * lines) {
    const int cnt = min(lines, npairs - g0);
    auto ld = [&](int l, int e) {
      const int z = div_magic(g0 + l, P.m_hy), y = 2 * (g0 + l - z * hy);
      const bool up = 2 * e > n;
      const int k = up ? n - e : e;
      const double2* row = in.at(z) + size_t(y) * P.nhp + k;
      const bool two = y + 1 < n;  // else the row again (no branch around a load)
      double2 a = row[0], b = row[two ? P.nhp : 0];
      if (!two) b = make_double2(0.0, 0.0);
      if (k == 0 || 2 * k == n) a.y = b.y = 0.0;  // real rows: rounding only
      if (up) {
        a.y = -a.y;
        b.y = -b.y;
      }
      return make_double2(a.y + b.x, a.x - b.y);
    };
    auto st = [&](int l, int e, double2 v) {
      const int z = div_magic(g0 + l, P.m_hy), y = 2 * (g0 + l - z * hy);
      sink.put(n, z, y, e, v.y);
      if (y + 1 < n) sink.put(n, z, y + 1, e, v.x);
    };
    fft_lines<NT, CLS, false>(P, M, cnt, buf, tw, ld, st);
    __syncthreads();
  }
}

// Complex columns along y (axis 1) or z (axis 2), from I to O (the same
// buffer: in place).  The inverse exchanges real and imaginary parts on the
// way in and out.
template <int NT, int CLS>
__global__ __launch_bounds__(NT, NT == 512 ? 4 : 3) void fft_columns_kernel(FftPlan P, ModeBuf I,
                                                         ModeBuf O,
                                                         const double2* __restrict__ twg, int lg,
                                                         int axis, int inverse) {
  extern __shared__ double2 smem[];
  const int n = P.n, L = 1 << lg, total = n * P.nhp;
  double2* tw = smem;
  double2* buf = smem + n;
  for (int i = int(threadIdx.x); i < n; i += NT) tw[i] = twg[i];
  const Modes in = modes_of(I, P), out = modes_of(O, P);
  const ColMap M{lg};
  __syncthreads();
  for (int g0 = int(blockIdx.x) * L; g0 < total; g0 += int(gridDim.x) * L) {
    // a thread works on one line of the group in every stage (L divides NT)
    const int id = g0 + (int(threadIdx.x) & (L - 1));
    const bool own = id < total;
    const int idc = own ? id : total - 1;
    const int z = div_magic(idc, P.m_nhp), x = idc - z * P.nhp;  // (z, kx) of a y line
    const double2* yin = in.at(axis == 1 ? z : 0) + x;
    double2* yout = out.at(axis == 1 ? z : 0) + x;
    auto ld = [&](int, int e) {
      const double2 v = axis == 1 ? yin[size_t(e) * P.nhp] : in.at(e)[idc];
      return inverse ? make_double2(v.y, v.x) : v;
    };
    auto st = [&](int, int e, double2 v) {
      if (own) (axis == 1 ? yout + size_t(e) * P.nhp : out.at(e) + idc)[0] = inverse ? make_double2(v.y, v.x) : v;
    };
    fft_lines<NT, CLS, false>(P, M, L, buf, tw, ld, st);
    __syncthreads();
  }
}

}  // namespace

// ---- host side --------------------------------------------------------------

FftPlan fft_plan(int n) {
  FftPlan P{};
  P.n = n;
  P.nh = n / 2 + 1;
  P.nhp = n >= 32 ? (P.nh + 7) / 8 * 8 : P.nh;
  int m = n, Ns = 1;
  auto add = [&](int r) {
    P.radix[P.nst] = r;
    P.ns[P.nst] = Ns;
    P.m_ns[P.nst] = magic_of(Ns);
    P.m_nr[P.nst] = magic_of(n / r);
    ++P.nst;
    Ns *= r;
    m /= r;
  };
  for (int r : {8, 4, 2, 7, 5, 3})
    while (m % r == 0) add(r);
  for (int r = 11; r <= m; r += 2)
    while (m % r == 0) {
      add(r);
      P.direct = 1;
    }
  // class: 0 only factors 8, 4, 2, 1 also 5 and 3, 2 anything else (7, larger
  // primes, and sides of a single stage, which class 2 passes through LDS)
  P.cls = P.nst < 2 ? 2 : 0;
  for (int k = 0; k < P.nst; ++k) {
    const int r = P.radix[k], c = r == 8 || r == 4 || r == 2 ? 0 : (r == 3 || r == 5 ? 1 : 2);
    if (c > P.cls) P.cls = c;
  }
  P.nt = n <= 256 ? 256 : 512;
  P.m_n = magic_of(n);
  P.m_nh = magic_of(P.nh);
  P.m_nhp = magic_of(P.nhp);
  P.m_hy = magic_of((n + 1) / 2);
  return P;
}

void fft_plan_unpad(FftPlan& P) {
  P.nhp = P.nh;
  P.m_nhp = magic_of(P.nhp);
}

int fft_column_lines_log2(const FftPlan& P) {
  const int most = P.nt * kFftPerThread / P.n;
  int lg = 0;
  while ((2 << lg) <= most && lg < 6) ++lg;
  // small lattices: fewer lines per group, to reach every CU (8 columns are
  // one 128-byte line)
  while (lg > 3 && (P.n * P.nhp >> lg) < 256) --lg;
  return lg;
}

size_t fft_lds_bytes(int n, int lines) {
  // the last value's padded place is below v + v/8.  Full groups of 2048
  // values of side 256 (4096 of side 512) take a quarter (half) of a CU's 160
  // KB to the byte.
  const size_t v = size_t(lines) * n;
  return (v + (v >> 3) + n) * sizeof(double2);
}

hipError_t launch_fft_tables(int n, const Stencil& st, double2* tw, double* ax, hipStream_t s) {
  hipLaunchKernelGGL(fft_tables_kernel, dim3((n + 255) / 256), dim3(256), 0, s, n, st, tw, ax);
  return hipGetLastError();
}

namespace {

// Groups of pairs of rows: small lattices take groups as small as it takes to
// reach every CU.
int row_lines(const FftPlan& P, int npairs) {
  int lines = P.nt * kFftPerThread / P.n;
  while (lines > 1 && npairs / lines < 256) lines = (lines + 1) / 2;
  return lines;
}

template <class Src>
hipError_t launch_r2c(const FftPlan& P, const Src& src, const ModeBuf& B, const double2* tw,
                      hipStream_t s) {
  const int n = P.n, npairs = n * ((n + 1) / 2), lines = row_lines(P, npairs);
  const int groups = (npairs + lines - 1) / lines;
  const dim3 grid(groups < kFftGridMax ? groups : kFftGridMax);
  const size_t lds = fft_lds_bytes(n, lines);
#define R2C_LAUNCH(NT, CLS) return fft_launch(r2c_rows_kernel<NT, CLS, Src>, grid, NT, lds, s, P, src, B, tw, lines, npairs)
  FFT_DISPATCH(P, R2C_LAUNCH);
#undef R2C_LAUNCH
}

template <class Sink>
hipError_t launch_c2r(const FftPlan& P, const ModeBuf& B, const Sink& sink, const double2* tw,
                      hipStream_t s) {
  const int n = P.n, npairs = n * ((n + 1) / 2), lines = row_lines(P, npairs);
  const int groups = (npairs + lines - 1) / lines;
  const dim3 grid(groups < kFftGridMax ? groups : kFftGridMax);
  const size_t lds = fft_lds_bytes(n, lines);
#define C2R_LAUNCH(NT, CLS) return fft_launch(c2r_rows_kernel<NT, CLS, Sink>, grid, NT, lds, s, P, B, sink, tw, lines, npairs)
  FFT_DISPATCH(P, C2R_LAUNCH);
#undef C2R_LAUNCH
}

template <typename T, bool MOMENTUM>
hipError_t r2c_lattice(const LatView& v, int field, const FftPlan& P, const ModeBuf& B,
                       const double2* tw, hipStream_t s) {
  LatticeRows<T, MOMENTUM> src;
  for (int k = 0; k < 2; ++k) {
    src.phi[k] = v.phi[k];
    src.pi[k] = v.pi[k];
  }
  src.sc = v.sc;
  src.zs = v.zs;
  src.field = field;
  return launch_r2c(P, src, B, tw, s);
}

}  // namespace

hipError_t launch_field_rows(const LatView& v, int field, int momentum, const FftPlan& P,
                             const ModeBuf& B, const double2* tw, hipStream_t s) {
  if (v.prec == SL_FP32)
    return momentum ? r2c_lattice<float, true>(v, field, P, B, tw, s)
                    : r2c_lattice<float, false>(v, field, P, B, tw, s);
  return momentum ? r2c_lattice<double, true>(v, field, P, B, tw, s)
                  : r2c_lattice<double, false>(v, field, P, B, tw, s);
}

hipError_t launch_fft_columns(const FftPlan& P, const ModeBuf& I, const ModeBuf& O, const double2* tw,
                              int axis, int inverse, hipStream_t s) {
  const int n = P.n, lg = fft_column_lines_log2(P), L = 1 << lg, groups = (n * P.nhp + L - 1) / L;
  const dim3 grid(groups < kFftGridMax ? groups : kFftGridMax);
  const size_t lds = fft_lds_bytes(n, L);
#define COL_LAUNCH(NT, CLS) return fft_launch(fft_columns_kernel<NT, CLS>, grid, NT, lds, s, P, I, O, tw, lg, axis, inverse)
  FFT_DISPATCH(P, COL_LAUNCH);
#undef COL_LAUNCH
}

hipError_t launch_rows_to_field(const LatView& v, int field, double base, double pi_value, const FftPlan& P,
                                const ModeBuf& B, const double2* tw, hipStream_t s) {
  if (v.prec == SL_FP32)
    return launch_c2r(P, B, LatticeSink<float>{v.phi[0], v.pi[0], v.zs, field, base, pi_value}, tw, s);
  return launch_c2r(P, B, LatticeSink<double>{v.phi[0], v.pi[0], v.zs, field, base, pi_value}, tw, s);
}

hipError_t launch_array_rows(const double* r, const double* shift, const FftPlan& P, const ModeBuf& B,
                             const double2* tw, hipStream_t s) {
  return launch_r2c(P, ArrayRows{r, shift}, B, tw, s);
}

hipError_t launch_rows_to_array(double* r, double scale, const double* add, const FftPlan& P,
                                const ModeBuf& B, const double2* tw, hipStream_t s) {
  return launch_c2r(P, B, ArraySink{r, scale, add}, tw, s);
}

}  // namespace symlat
