// Observables and state exchange: lattice sums for eq. (2.16), (2.18),
// (2.20), (3.1) at the synchronised state, the constraint solve for p_a, the
// momentum sum S2, and FP64 export/import of the fields.

#include "device.h"

namespace symlat {

namespace {

constexpr int kDiagBlocksMax = 1024;
// target tile count of the observables passes: two tiles per CU
// (measured at 256^3, 7-point: 1024 tiles took 4-13 % longer; a tile
// writes 2 nsums doubles of partials and the buffer holds 4096 tiles of
// the largest count, the most that n = 1024 makes)
constexpr int kDiagTiles = 512;

// Compile-time index of one of two register sets.
template <int I>
struct Half {
  static constexpr int value = I;
};

struct Bufs {
  const void* phi[2];
  const void* pi[2];
};

Bufs bufs_of(const LatView& v) {
  Bufs B;
  for (int k = 0; k < 2; ++k) {
    B.phi[k] = v.phi[k];
    B.pi[k] = v.pi[k];
  }
  return B;
}

// Per-field sums then the potential: [pi^2, G, phi-s, (phi-s)^2, phi D phi] * NF, V
template <int NF>
constexpr int nsums() { return 5 * NF + 1; }

// The sums for the 7-point stencil, walked like the fused pass: a
// workgroup owns a column tile (one wavefront per row, VX sites per lane) and
// marches tz planes up in z.  Plane z goes to LDS (double-buffered, one barrier
// per plane) with the row above the tile and the column right of it, which
// designated lanes load.  Each bond is visited once, from its lower end: over
// the periodic lattice sum_x G = sum of (f(x + e) - f(x))^2 over the three
// forward neighbours, and sum_x f D f = -sum_x G, so neither the other three
// neighbours nor D are formed (and f D f, whose terms are of the order of f^2
// times a rounding error, is not summed).  The kernel is bound by
// instructions: with all six neighbours and D a read-out took 196 us at 256^3
// in FP64 with two fields and 143 us in FP32, whatever the loads' distance; now
// 138 and 92 us (about 23 us of each is the launches and the wait; before, 40),
// and 1025 -> 803 us at 512^3 q-ball.
// The loads run two planes ahead of the arithmetic, in two register sets used
// in turn.  A lane adds each of its sites' terms plainly over the chunk, and the
// sites', lanes' and tiles' totals are combined with compensation (both sites in
// one sum were 2.6e-14 of the total off at 512^3, where one site's are 5e-16; the
// second set of sums costs no time).
constexpr int kEX = 64, kEY = kBlock / kEX;

template <typename T, int VX>
struct SiteVec {
  double v[VX];
};

template <typename T, int VX>
__device__ __forceinline__ SiteVec<T, VX> load_sites(const T* __restrict__ p) {
  static_assert(VX == 1 || sizeof(T) == 8, "");
  SiteVec<T, VX> r;
  if constexpr (VX == 1) {
    r.v[0] = double(p[0]);
  } else {
    const double2 q = *reinterpret_cast<const double2*>(p);
    r.v[0] = q.x;
    r.v[1] = q.y;
  }
  return r;
}

template <typename T, int NF, int KIND, int VX>
__global__ __launch_bounds__(kBlock) void energies7_kernel(Bufs B, const DevScalars* sc,
                                                          PotArgs prm, int n, int zs, int tz,
                                                          double* partials) {
  constexpr int NV = nsums<NF>();
  constexpr int W = kEX * VX, LW = W + VX;  // sites of a tile row; LDS row
  __shared__ KSum scratch[4 * NV];
  __shared__ double lds[2][NF][LW * (kEY + 1)];
  const int par = sc->parity;
  const T* __restrict__ phi = static_cast<const T*>(B.phi[par]);
  const T* __restrict__ pi = static_cast<const T*>(B.pi[par]);
  const double c = sc->c_pend;
  PotT<double> pot;
#pragma unroll
  for (int i = 0; i < kMaxFields; ++i) pot.p[i] = prm.p[i];
  const size_t n2 = size_t(n) * n;
  // offsets of the stored remainders (0 in FP64 storage), drifted by c
  double offp[NF], offq[NF], shift[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    offq[i] = sc->off_pi[i];
    offp[i] = sc->off_phi[i] + c * offq[i];
    shift[i] = offp[i] + fma(c, double(pi[i * n2]), double(phi[i * n2]));
  }

  const int ntx = (n + W - 1) / W, nty = (n + kEY - 1) / kEY;
  int b = blockIdx.x;
  const int xt = b % ntx;
  b /= ntx;
  const int yt = b % nty;
  const int zt = b / nty;
  const int x0 = xt * W, y0 = yt * kEY, z0 = zt * tz;
  const int wx = min(W, n - x0), wy = min(kEY, n - y0), zend = min(z0 + tz, n);
  const int tid = int(threadIdx.x), tx = tid % kEX, ty = tid / kEX;
  const bool active = tx * VX < wx && ty < wy;
  const int own = ty * LW + tx * VX;
  // every lane issues the same loads (idle lanes read the tile's first
  // column, in range and unused), so that no branch around them makes the
  // compiler wait for the loads in flight
  const unsigned r = active ? unsigned(y0 + ty) * n + (x0 + tx * VX) : unsigned(y0) * n + x0;

  // halo job: the row above (VX sites), the column right of the tile (the
  // first site of its group; VX divides n)
  int hjob = 0, hl = 0;
  unsigned hr = r;
  if (tid < kEX) {
    if (tid * VX < wx) {
      hjob = VX;
      hr = unsigned(y0 + wy == n ? 0 : y0 + wy) * n + x0 + tid * VX;
      hl = wy * LW + tid * VX;
    }
  } else if (tid < kEX + kEY) {
    const int q = tid - kEX;
    if (q < wy) {
      hjob = 1;
      hr = unsigned(y0 + q) * n + (x0 + wx == n ? 0 : x0 + wx);
      hl = q * LW + wx;
    }
  }

  auto wrapz = [n](int zz) { return zz >= n ? zz - n : zz; };
  double part[VX][NV];  // of the lane's first and second sites
#pragma unroll
  for (int v = 0; v < VX; ++v)
#pragma unroll
    for (int k = 0; k < NV; ++k) part[v][k] = 0.0;
  // drifted field at z, z+1 and momenta at z of the own sites; drifted halo
  // of plane z
  double fc[NF][VX], fp[NF][VX], pc[NF][VX], pp[NF][VX], hc[NF][VX];
  // loads in flight: remainders and momenta of the own sites and the halo
  struct Flight {
    SiteVec<T, VX> f[NF], p[NF], h[NF], q[NF];
  };
  auto load_own = [&](int zz, Flight& F) {
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      const size_t o = (size_t(zz) * zs + i) * n2;
      F.f[i] = load_sites<T, VX>(phi + o + r);
      F.p[i] = load_sites<T, VX>(pi + o + r);
    }
  };
  auto load_halo = [&](int zz, Flight& F) {
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      const size_t o = (size_t(zz) * zs + i) * n2;
      F.h[i] = load_sites<T, VX>(phi + o + hr);
      F.q[i] = load_sites<T, VX>(pi + o + hr);
    }
  };
  auto take_own = [&](const Flight& F) {
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int v = 0; v < VX; ++v) {
        fp[i][v] = offp[i] + fma(c, F.p[i].v[v], F.f[i].v[v]);
        pp[i][v] = offq[i] + F.p[i].v[v];
      }
  };
  auto take_halo = [&](const Flight& F) {
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int v = 0; v < VX; ++v) hc[i][v] = offp[i] + fma(c, F.q[i].v[v], F.h[i].v[v]);
  };
  auto shift_planes = [&]() {
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int v = 0; v < VX; ++v) {
        fc[i][v] = fp[i][v];
        pc[i][v] = pp[i][v];
      }
  };
  Flight fl[2];
  // loads of own plane zz + 2 and halo plane zz + 1; past the chunk end they
  // re-read the last planes (in range, unused)
  auto issue = [&](int zz, Flight& F) {
    load_own(wrapz(min(zz + 2, zend)), F);
    load_halo(min(zz + 1, zend - 1), F);
  };
  load_own(z0, fl[0]);
  load_halo(z0, fl[0]);
  load_own(wrapz(z0 + 1), fl[1]);
  take_own(fl[0]);
  take_halo(fl[0]);
  shift_planes();
  issue(z0, fl[0]);
  take_own(fl[1]);
  // plane z: the next plane's loads go out into the other set, this plane's
  // (set H) are taken at the end
  auto plane = [&](auto set, int z) {
    constexpr int H = decltype(set)::value;
    issue(z + 1, fl[1 - H]);
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      if (active) {
#pragma unroll
        for (int v = 0; v < VX; ++v) lds[H][i][own + v] = fc[i][v];
      }
      if (hjob == VX) {
#pragma unroll
        for (int v = 0; v < VX; ++v) lds[H][i][hl + v] = hc[i][v];
      } else if (hjob) {
        lds[H][i][hl] = hc[i][0];
      }
    }
    __syncthreads();
    if (active) {
#pragma unroll
      for (int v = 0; v < VX; ++v) {
        double f[NF];
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          const double* L = lds[H][i] + own + v;
          const double fcv = fc[i][v];
          const double dx = (v + 1 < VX ? fc[i][v + 1 < VX ? v + 1 : v] : L[1]) - fcv;
          const double dy = L[LW] - fcv, dz = fp[i][v] - fcv;
          part[v][5 * i + 0] = fma(pc[i][v], pc[i][v], part[v][5 * i + 0]);
          part[v][5 * i + 1] += fma(dx, dx, fma(dy, dy, dz * dz));
          const double ds = fcv - shift[i];
          part[v][5 * i + 2] += ds;
          part[v][5 * i + 3] = fma(ds, ds, part[v][5 * i + 3]);
          f[i] = fcv;
        }
        double V, dV[NF];
        potential<KIND, NF, double>(f, pot, V, dV);
        part[v][5 * NF] += V;
      }
    }
    shift_planes();
    take_own(fl[H]);
    take_halo(fl[H]);
  };
  int z = z0;
  for (; z + 1 < zend; z += 2) {
    plane(Half<0>{}, z);
    plane(Half<1>{}, z + 1);
  }
  if (z < zend) plane(Half<0>{}, z);
#pragma unroll
  for (int v = 0; v < VX; ++v)
#pragma unroll
    for (int i = 0; i < NF; ++i) part[v][5 * i + 4] = -part[v][5 * i + 1];
  KSum acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    acc[k] = KSum{part[0][k], 0.0};
#pragma unroll
    for (int v = 1; v < VX; ++v) kadd(acc[k], part[v][k]);
  }
  block_reduce<NV>(acc, scratch);
  if (threadIdx.x == 0) {
    double* out = partials + size_t(blockIdx.x) * 2 * NV;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      out[2 * k] = acc[k].s;
      out[2 * k + 1] = acc[k].c;
    }
  }
}

// The sums with a general member of the cubic family, walked the same way with
// one site per lane: 13 forward neighbours stand for the 26, four in the plane
// and nine in the next, so a plane goes to LDS with a whole ring of halo cells
// and three planes are kept (one barrier per plane).  With
// G = 1/2 sum_d c_d (f(x + d) - f(x))^2 and D f = sum_d c_d (f(x + d) - f(x))
// + rest f, rest = c0 + 6 c1 + 12 c2 + 8 c3 (0 up to rounding),
// sum_x f D f = -sum_x G + rest sum_x f^2.  Every term is added with
// compensation: 128 planes of a homogeneous state added plainly were 3.4e-15 of
// the total off, now less than 3e-16.  It is bound by instructions and LDS reads:
// a read-out takes 188 us at 256^3 in FP64 with two fields and 156 in FP32 (184
// and 135 with plain sums); with each site reading 26 neighbours and their
// momenta from memory it took 1053 and 591 us.
template <typename T, int NF, int KIND>
__global__ __launch_bounds__(kBlock) void energies27_kernel(Bufs B, const DevScalars* sc,
                                                           PotArgs prm, int n, int zs, int tz,
                                                           Stencil st, double* partials) {
  constexpr int NV = nsums<NF>();
  constexpr int LX = kEX + 2, P = LX * (kEY + 2);
  static_assert(2 * kEX + 2 * kEY + 4 <= kBlock, "one halo cell per thread");
  __shared__ KSum scratch[4 * NV];
  extern __shared__ double planes[];  // [3][NF][P]
  const int par = sc->parity;
  const T* __restrict__ phi = static_cast<const T*>(B.phi[par]);
  const T* __restrict__ pi = static_cast<const T*>(B.pi[par]);
  const double c = sc->c_pend;
  PotT<double> pot;
#pragma unroll
  for (int i = 0; i < kMaxFields; ++i) pot.p[i] = prm.p[i];
  const size_t n2 = size_t(n) * n;
  // offsets of the stored remainders (0 in FP64 storage), drifted by c
  double offp[NF], offq[NF], shift[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    offq[i] = sc->off_pi[i];
    offp[i] = sc->off_phi[i] + c * offq[i];
    shift[i] = offp[i] + fma(c, double(pi[i * n2]), double(phi[i * n2]));
  }

  const int ntx = (n + kEX - 1) / kEX, nty = (n + kEY - 1) / kEY;
  int b = blockIdx.x;
  const int xt = b % ntx;
  b /= ntx;
  const int yt = b % nty, zt = b / nty;
  const int x0 = xt * kEX, y0 = yt * kEY, z0 = zt * tz;
  const int wx = min(kEX, n - x0), wy = min(kEY, n - y0), zend = min(z0 + tz, n);
  const int tid = int(threadIdx.x), tx = tid % kEX, ty = tid / kEX;
  const bool active = tx < wx && ty < wy;
  const int own = (ty + 1) * LX + 1 + tx;
  // every lane issues the same loads (see above)
  const unsigned r = active ? unsigned(y0 + ty) * n + (x0 + tx) : unsigned(y0) * n + x0;

  // halo job: one cell of the ring around the tile
  int hl = -1;
  unsigned hr = r;
  {
    const int xl = x0 == 0 ? n - 1 : x0 - 1, xr = x0 + wx == n ? 0 : x0 + wx;
    const int yl = y0 == 0 ? n - 1 : y0 - 1, yr = y0 + wy == n ? 0 : y0 + wy;
    int hx = 0, hy = 0;
    if (tid < 2 * kEX) {
      const bool up = tid >= kEX;
      const int t = up ? tid - kEX : tid;
      if (t < wx) {
        hx = x0 + t;
        hy = up ? yr : yl;
        hl = (up ? wy + 1 : 0) * LX + 1 + t;
      }
    } else if (tid < 2 * kEX + 2 * kEY) {
      const int q = tid - 2 * kEX;
      const bool right = q >= kEY;
      const int t = right ? q - kEY : q;
      if (t < wy) {
        hx = right ? xr : xl;
        hy = y0 + t;
        hl = (t + 1) * LX + (right ? wx + 1 : 0);
      }
    } else if (tid < 2 * kEX + 2 * kEY + 4) {
      const int q = tid - 2 * kEX - 2 * kEY;
      hx = (q & 1) ? xr : xl;
      hy = (q & 2) ? yr : yl;
      hl = ((q & 2) ? wy + 1 : 0) * LX + ((q & 1) ? wx + 1 : 0);
    }
    if (hl >= 0) hr = unsigned(hy) * n + hx;
  }

  auto wrapz = [n](int zz) { return zz >= n ? zz - n : zz; };
  KSum acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = KSum{0.0, 0.0};
  double fc[NF], pc[NF], fn[NF], pn[NF];  // own site at z and z + 1
  T lf[NF], lp[NF], hf[NF], hp[NF];       // loads in flight: own site, halo cell
  auto issue = [&](int zz) {
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      const size_t o = (size_t(zz) * zs + i) * n2;
      lf[i] = phi[o + r];
      lp[i] = pi[o + r];
      hf[i] = phi[o + hr];
      hp[i] = pi[o + hr];
    }
  };
  // the plane in flight to LDS buffer k, its own site to fn and pn
  auto land = [&](int k) {
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      double* L = planes + size_t(k * NF + i) * P;
      fn[i] = offp[i] + fma(c, double(lp[i]), double(lf[i]));
      pn[i] = offq[i] + double(lp[i]);
      if (active) L[own] = fn[i];
      if (hl >= 0) L[hl] = offp[i] + fma(c, double(hp[i]), double(hf[i]));
    }
  };
  auto next = [&]() {
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      fc[i] = fn[i];
      pc[i] = pn[i];
    }
  };
  issue(z0);
  land(0);
  next();
  issue(wrapz(z0 + 1));
  int k0 = 0, count = 0;
  for (int z = z0; z < zend; ++z) {
    const int k1 = k0 == 2 ? 0 : k0 + 1;
    land(k1);
    __syncthreads();
    issue(wrapz(min(z + 2, zend)));  // past the chunk's end: in range, unused
    if (active) {
      ++count;
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        const double* A = planes + size_t(k0 * NF + i) * P + own;
        const double* U = planes + size_t(k1 * NF + i) * P + own;
        const double f = fc[i];
        auto sq = [f](double v, double s) {
          const double d = v - f;
          return fma(d, d, s);
        };
        const double faces = sq(fn[i], sq(A[LX], sq(A[1], 0.0)));
        const double edges = sq(U[LX], sq(U[-LX], sq(U[1], sq(U[-1], sq(A[LX + 1], sq(A[LX - 1], 0.0))))));
        const double corners = sq(U[LX + 1], sq(U[LX - 1], sq(U[-LX + 1], sq(U[-LX - 1], 0.0))));
        kadd(acc[5 * i + 0], pc[i] * pc[i]);
        kadd(acc[5 * i + 1], fma(st.c[1], faces, fma(st.c[2], edges, st.c[3] * corners)));
        const double ds = f - shift[i];
        kadd(acc[5 * i + 2], ds);
        kadd(acc[5 * i + 3], ds * ds);
      }
      double V, dV[NF];
      potential<KIND, NF, double>(fc, pot, V, dV);
      kadd(acc[5 * NF], V);
    }
    next();
    k0 = k1;
  }
  const double rest = (st.c[0] + 6.0 * st.c[1]) + (12.0 * st.c[2] + 8.0 * st.c[3]);
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const double m1 = acc[5 * i + 2].s + acc[5 * i + 2].c, m2 = acc[5 * i + 3].s + acc[5 * i + 3].c;
    const double f2 = m2 + shift[i] * (2.0 * m1 + shift[i] * count);
    acc[5 * i + 4] = KSum{-acc[5 * i + 1].s, -acc[5 * i + 1].c};
    kadd(acc[5 * i + 4], rest * f2);
  }
  block_reduce<NV>(acc, scratch);
  if (threadIdx.x == 0) {
    double* out = partials + size_t(blockIdx.x) * 2 * NV;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      out[2 * k] = acc[k].s;
      out[2 * k + 1] = acc[k].c;
    }
  }
}

// Reduce energies partials, compute observables; mode 1 also solves the
// constraint H = 0 for p_a (expanding branch) and sets S2.  In mode 0 the
// scalars follow the observables, so that one place holds what a call returns.
template <int NF>
__global__ __launch_bounds__(kBlock) void energies_finalize(const double* partials, int nblocks,
                                                           DevScalars* sc, BgConsts K, int n,
                                                           Bufs B, int prec, double* sums_out,
                                                           sl_energies_t* out, int mode) {
  constexpr int NV = nsums<NF>();
  __shared__ KSum scratch[4 * NV];
  // the scalars and the sums' shift (phi_sync at site 0) are in flight while
  // the partials are reduced
  DevScalars S = *sc;
  double sh[NF];
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    const size_t o = size_t(i) * n * n;
    const double offp = S.off_phi[i] + S.c_pend * S.off_pi[i];
    const void *ph = B.phi[S.parity], *pp = B.pi[S.parity];
    sh[i] = prec == SL_FP32
                ? offp + fma(S.c_pend, double(static_cast<const float*>(pp)[o]), double(static_cast<const float*>(ph)[o]))
                : offp + fma(S.c_pend, static_cast<const double*>(pp)[o], static_cast<const double*>(ph)[o]);
  }
  KSum v[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = KSum{0.0, 0.0};
  for (int b = threadIdx.x; b < nblocks; b += kBlock) {
    const double* p = partials + size_t(b) * 2 * NV;
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = kcombine(v[k], KSum{p[2 * k], p[2 * k + 1]});
  }
  // a wavefront per quarter of the rows, then one thread per sum
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = wave_reduce(v[k]);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) scratch[(threadIdx.x >> 6) * NV + k] = v[k];
  }
  __syncthreads();
  __shared__ double s[NV];
  if (threadIdx.x < NV) {
    KSum t = scratch[threadIdx.x];
#pragma unroll
    for (int w = 1; w < kBlock / 64; ++w) t = kcombine(t, scratch[w * NV + threadIdx.x]);
    s[threadIdx.x] = t.s + t.c;
    sums_out[threadIdx.x] = s[threadIdx.x];
  }
  __syncthreads();
  // the scalars behind a read-out (mode 0 leaves them as they are)
  constexpr int kWords = int(sizeof(DevScalars) / sizeof(uint64_t));
  static_assert(kWords <= 64 && sizeof(sl_energies_t) % sizeof(uint64_t) == 0, "whole words");
  if (mode == 0 && threadIdx.x >= 64 && threadIdx.x < 64 + kWords)
    reinterpret_cast<uint64_t*>(out + 1)[threadIdx.x - 64] = reinterpret_cast<const uint64_t*>(sc)[threadIdx.x - 64];
  if (threadIdx.x != 0) return;
  const double VL = K.VL;
  const double a = S.a;
  const double a2 = a * a, a4 = a2 * a2, a6 = a4 * a2;
  sl_energies_t E;
  for (int i = 0; i < 8; ++i) E.kin[i] = E.grad[i] = E.mean[i] = E.var[i] = 0.0;
  double S2 = 0.0, SdD = 0.0, skin = 0.0, sgrad = 0.0;
#pragma unroll
  for (int i = 0; i < NF; ++i) {
    E.kin[i] = (s[5 * i] / VL) / (2.0 * a6);
    E.grad[i] = (s[5 * i + 1] / VL) / (2.0 * a2 * K.dx2);
    const double m1 = s[5 * i + 2] / VL;
    E.mean[i] = sh[i] + m1;
    E.var[i] = s[5 * i + 3] / VL - m1 * m1;
    S2 += s[5 * i];
    SdD += s[5 * i + 4];
    skin += E.kin[i];
    sgrad += E.grad[i];
  }
  const double SV = s[5 * NF];
  E.pot = SV / VL;
  E.rho = skin + sgrad + E.pot;
  E.pressure = skin - sgrad / 3.0 - E.pot;
  E.w_eos = E.rho != 0.0 ? E.pressure / E.rho : __builtin_nan("");
  // field part of eq. (2.20) plus the radiation and matter terms
  const double Hf = S2 / (2.0 * a2) - a2 * SdD / (2.0 * K.dx2) + a4 * SV;
  const double Hext = K.VL_rho_r + a * K.VL_rho_m;
  if (mode == 1) {
    S.S2 = S2;
    if (K.expand) {
      const double E0 = Hf + Hext;
      if (E0 >= 0.0) {
        S.p_a = -sqrt(12.0 * VL * K.mpl2 * E0);
      } else {
        S.p_a = __builtin_nan("");
        S.status |= kStatusNonFinite;
      }
    } else {
      S.p_a = 0.0;
    }
    *sc = S;
  }
  E.eta = S.eta;
  E.a = a;
  E.p_a = S.p_a;
  if (K.expand) {
    E.hubble = -S.p_a / (6.0 * VL * K.mpl2 * a2);
    const double rho_tot = E.rho + (K.VL_rho_r / VL) / a4 + (K.VL_rho_m / VL) / (a2 * a);
    E.friedmann_residual = fabs(rho_tot / (3.0 * K.mpl2 * E.hubble * E.hubble) - 1.0);
    E.h_total = -S.p_a * S.p_a / (12.0 * VL * K.mpl2) + Hf + Hext;
  } else {
    E.hubble = 0.0;
    E.friedmann_residual = __builtin_nan("");
    E.h_total = Hf + Hext;
  }
  *out = E;
}

template <typename T, int NF, int KIND>
hipError_t energies_t(const LatView& v, double* sums, sl_energies_t* out, int mode, hipStream_t s) {
  const Bufs B = bufs_of(v);
  // z-chunks so that the tiles number about kDiagTiles (at most one chunk
  // per plane).  Two sites per lane in FP64 where rows divide, with up to
  // two fields (registers): 157 us a call at 256^3 with two fields against
  // 172 (both with the former read-back, some 17 us more); in FP32, where a
  // lane's load stays short of 16 bytes, one site is as fast or faster (111
  // against 114 us there, 835 against 874 at 512^3 q-ball)
  const int vx = v.st.kind == 0 && sizeof(T) == 8 && NF <= 2 && v.n % 2 == 0 ? 2 : 1;
  const int cols = ((v.n + kEX * vx - 1) / (kEX * vx)) * ((v.n + kEY - 1) / kEY);
  int ntz = kDiagTiles / cols;
  ntz = ntz < 1 ? 1 : (ntz > v.n ? v.n : ntz);
  const int tz = (v.n + ntz - 1) / ntz, nb = cols * ((v.n + tz - 1) / tz);
  if (v.st.kind != 0) {
    const size_t lds = size_t(3) * NF * (kEX + 2) * (kEY + 2) * sizeof(double);
    if (lds > 65536) {  // above 64 KB a kernel has to be told
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(energies27_kernel<T, NF, KIND>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((energies27_kernel<T, NF, KIND>), dim3(nb), dim3(kBlock), lds, s, B, v.sc,
                       v.prm, v.n, v.zs, tz, v.st, v.partials);
  } else if (vx == 2) {
    if constexpr (sizeof(T) == 8 && NF <= 2)
      hipLaunchKernelGGL((energies7_kernel<T, NF, KIND, 2>), dim3(nb), dim3(kBlock), 0, s, B, v.sc,
                         v.prm, v.n, v.zs, tz, v.partials);
  } else {
    hipLaunchKernelGGL((energies7_kernel<T, NF, KIND, 1>), dim3(nb), dim3(kBlock), 0, s, B, v.sc,
                       v.prm, v.n, v.zs, tz, v.partials);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((energies_finalize<NF>), dim3(1), dim3(kBlock), 0, s, v.partials, nb, v.sc,
                     v.bg, v.n, B, v.prec, sums, out, mode);
  return hipGetLastError();
}

template <typename T>
hipError_t energies_dispatch(const LatView& v, double* sums, sl_energies_t* out, int mode,
                             hipStream_t s) {
  switch (v.pot) {
    case SL_POT_CHAOTIC2: return energies_t<T, 2, SL_POT_CHAOTIC2>(v, sums, out, mode, s);
    case SL_POT_OSCILLON: return energies_t<T, 1, SL_POT_OSCILLON>(v, sums, out, mode, s);
    case SL_POT_QBALL_LOG: return energies_t<T, 2, SL_POT_QBALL_LOG>(v, sums, out, mode, s);
    default: break;
  }
  switch (v.nf) {
    case 1: return energies_t<T, 1, SL_POT_FREE>(v, sums, out, mode, s);
    case 2: return energies_t<T, 2, SL_POT_FREE>(v, sums, out, mode, s);
    case 3: return energies_t<T, 3, SL_POT_FREE>(v, sums, out, mode, s);
    case 4: return energies_t<T, 4, SL_POT_FREE>(v, sums, out, mode, s);
    case 5: return energies_t<T, 5, SL_POT_FREE>(v, sums, out, mode, s);
    case 6: return energies_t<T, 6, SL_POT_FREE>(v, sums, out, mode, s);
    case 7: return energies_t<T, 7, SL_POT_FREE>(v, sums, out, mode, s);
    case 8: return energies_t<T, 8, SL_POT_FREE>(v, sums, out, mode, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void sum_pi2_kernel(Bufs B, const DevScalars* sc,
                                                        size_t count, size_t n3, size_t n2, int zs,
                                                        double* partials) {
  __shared__ KSum scratch[4];
  const T* __restrict__ pi = static_cast<const T*>(B.pi[sc->parity]);
  KSum acc[1] = {{0.0, 0.0}};
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < count; e += stride) {
    const size_t i = e / n3;  // field i, site e - i n^3
    const double p = sc->off_pi[i] + double(pi[field_site(int(i), e - i * n3, zs, n2)]);
    kadd(acc[0], p * p);
  }
  block_reduce<1>(acc, scratch);
  if (threadIdx.x == 0) {
    partials[2 * blockIdx.x] = acc[0].s;
    partials[2 * blockIdx.x + 1] = acc[0].c;
  }
}

__global__ __launch_bounds__(kBlock) void sum_pi2_finalize(const double* partials, int nblocks,
                                                          DevScalars* sc) {
  __shared__ KSum scratch[4];
  KSum v[1] = {{0.0, 0.0}};
  for (int b = threadIdx.x; b < nblocks; b += kBlock)
    v[0] = kcombine(v[0], KSum{partials[2 * b], partials[2 * b + 1]});
  block_reduce<1>(v, scratch);
  if (threadIdx.x == 0) {
    const double S2 = v[0].s + v[0].c;
    sc->S2 = S2;
    if (!dev_finite(S2)) sc->status |= kStatusNonFinite;
  }
}

// Device offset of host element e: the host arrays are [field][z][y][x].
__device__ __forceinline__ size_t device_index(size_t e, int zs, size_t n2, size_t n3) {
  const size_t i = e / n3;
  return field_site(int(i), e - i * n3, zs, n2);
}

template <typename T>
__global__ void export_kernel(Bufs B, const DevScalars* sc, size_t count, int nf, int zs,
                              size_t n2, double* phi_out, double* pi_out) {
  const int par = sc->parity;
  const T* __restrict__ phi = static_cast<const T*>(B.phi[par]);
  const T* __restrict__ pi = static_cast<const T*>(B.pi[par]);
  const double c = sc->c_pend;
  const size_t n3 = count / nf;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < count; e += stride) {
    const size_t d = device_index(e, zs, n2, n3);
    const size_t i = e / n3;
    const double pr = double(pi[d]);
    if (phi_out) phi_out[e] = (sc->off_phi[i] + c * sc->off_pi[i]) + fma(c, pr, double(phi[d]));
    if (pi_out) pi_out[e] = sc->off_pi[i] + pr;
  }
}

template <typename T>
__global__ void import_kernel(void* phi0, void* pi0, size_t count, int nf, int zs, size_t n2,
                              const double* phi_in, const double* pi_in, Offsets off) {
  T* __restrict__ phi = static_cast<T*>(phi0);
  T* __restrict__ pi = static_cast<T*>(pi0);
  const size_t n3 = count / nf;
  const size_t stride = size_t(gridDim.x) * blockDim.x;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < count; e += stride) {
    const size_t d = device_index(e, zs, n2, n3);
    const size_t i = e / n3;
    phi[d] = static_cast<T>(phi_in[e] - off.phi[i]);
    pi[d] = static_cast<T>(pi_in[e] - off.pi[i]);
  }
}

// One record per batch member, in table order, for a single read-back.
__global__ void gather_scalars_kernel(const BatchRun* __restrict__ runs, int nruns,
                                      DevScalars* __restrict__ out) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < nruns) out[r] = *runs[r].sc[0];
}

__global__ void reset_scalars_kernel(DevScalars* sc, double a, double p_a, Offsets off) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    DevScalars S = *sc;  // keeps the history buffer; a reset restarts it
    for (int i = 0; i < kMaxFields; ++i) {
      S.off_phi[i] = off.phi[i];
      S.off_pi[i] = off.pi[i];
    }
    S.a = a;
    S.p_a = p_a;
    S.eta = 0.0;
    S.S2 = 0.0;
    S.c_pend = 0.0;
    S.c_next = 0.0;
    S.alpha = 0.0;
    S.beta = 0.0;
    S.a_kick = a;
    S.S3_last = 0.0;
    S.parity = 0;
    S.status = 0;
    S.hist_n = 0;
    *sc = S;
  }
}

int grid_for(size_t count) {
  size_t nb = (count + kBlock - 1) / kBlock;
  if (nb > 4096) nb = 4096;
  if (nb < 1) nb = 1;
  return int(nb);
}

}  // namespace

hipError_t launch_energies(const LatView& v, double* sums, sl_energies_t* out, int mode,
                           hipStream_t s) {
  return v.prec == SL_FP32 ? energies_dispatch<float>(v, sums, out, mode, s)
                           : energies_dispatch<double>(v, sums, out, mode, s);
}

hipError_t launch_sum_pi2(const LatView& v, hipStream_t s) {
  const size_t count = size_t(v.nf) * v.n * v.n * v.n;
  const int nb = grid_for(count) > kDiagBlocksMax ? kDiagBlocksMax : grid_for(count);
  const Bufs B = bufs_of(v);
  if (v.prec == SL_FP32)
    hipLaunchKernelGGL(sum_pi2_kernel<float>, dim3(nb), dim3(kBlock), 0, s, B, v.sc, count,
                       count / v.nf, size_t(v.n) * v.n, v.zs, v.partials);
  else
    hipLaunchKernelGGL(sum_pi2_kernel<double>, dim3(nb), dim3(kBlock), 0, s, B, v.sc, count,
                       count / v.nf, size_t(v.n) * v.n, v.zs, v.partials);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sum_pi2_finalize, dim3(1), dim3(kBlock), 0, s, v.partials, nb, v.sc);
  return hipGetLastError();
}

hipError_t launch_export(const LatView& v, double* phi_out, double* pi_out, hipStream_t s) {
  const size_t count = size_t(v.nf) * v.n * v.n * v.n;
  const Bufs B = bufs_of(v);
  if (v.prec == SL_FP32)
    hipLaunchKernelGGL(export_kernel<float>, dim3(grid_for(count)), dim3(kBlock), 0, s, B, v.sc,
                       count, v.nf, v.zs, size_t(v.n) * v.n, phi_out, pi_out);
  else
    hipLaunchKernelGGL(export_kernel<double>, dim3(grid_for(count)), dim3(kBlock), 0, s, B, v.sc,
                       count, v.nf, v.zs, size_t(v.n) * v.n, phi_out, pi_out);
  return hipGetLastError();
}

hipError_t launch_import(const LatView& v, const double* phi_in, const double* pi_in, double a,
                         double p_a, const Offsets& off, hipStream_t s) {
  const size_t count = size_t(v.nf) * v.n * v.n * v.n;
  if (v.prec == SL_FP32)
    hipLaunchKernelGGL(import_kernel<float>, dim3(grid_for(count)), dim3(kBlock), 0, s, v.phi[0],
                       v.pi[0], count, v.nf, v.zs, size_t(v.n) * v.n, phi_in, pi_in, off);
  else
    hipLaunchKernelGGL(import_kernel<double>, dim3(grid_for(count)), dim3(kBlock), 0, s, v.phi[0],
                       v.pi[0], count, v.nf, v.zs, size_t(v.n) * v.n, phi_in, pi_in, off);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(reset_scalars_kernel, dim3(1), dim3(64), 0, s, v.sc, a, p_a, off);
  return hipGetLastError();
}

hipError_t launch_gather_scalars(const BatchRun* runs_dev, int nruns, DevScalars* out_dev,
                                 hipStream_t s) {
  if (nruns <= 0) return hipSuccess;
  hipLaunchKernelGGL(gather_scalars_kernel, dim3((nruns + 255) / 256), dim3(256), 0, s, runs_dev,
                     nruns, out_dev);
  return hipGetLastError();
}

hipError_t launch_reset_scalars(const LatView& v, double a, double p_a, const Offsets& off,
                                hipStream_t s) {
  hipLaunchKernelGGL(reset_scalars_kernel, dim3(1), dim3(64), 0, s, v.sc, a, p_a, off);
  return hipGetLastError();
}

}  // namespace symlat
