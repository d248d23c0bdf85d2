// Level synchronisation kernels for gfx950: coarse/fine registers, reflux,
// EMF correction and restriction (the (S)ynchronise and (R)estrict steps of
// the paper's level cycle, Sec. 4).  Every kernel is a gather over tables
// built by the host runtime: one thread per register, cell or face copy, so
// each output has exactly one writer and no atomics are used.
#include "amr_internal.hpp"
#include "emf.hpp"
#include "sync_internal.hpp"

namespace amr {

namespace {

inline int blocks_for(int64_t n) {
  int64_t b = (n + 255) / 256;
  if (b > 65535) b = 65535;
  return (int)(b < 1 ? 1 : b);
}

// The refinement ratio of a synchronised hierarchy (the runtime refuses any
// other): the gathers below are unrolled over it, so each thread issues all
// of its loads before the first use and sums them in the order the
// definition states (one memory latency per thread instead of one per term).
constexpr int kR = 2;

// 1 / n of the n faces or edges a register averages: a power of the ratio,
// so the product with it is the quotient, to the bit.
template <class T> __device__ __forceinline__ T inv_count(int n) { return n == 1 ? T(1) : n == 2 ? T(0.5) : T(0.25); }

// One face register: the cell-updating flux components at each of its faces,
// all loads issued before the first use.  Component c of direction d carries
// lab slot 1 + (c - 1 + d) mod 3 of the momenta, 2-D's cell field is component
// 6 along x and 5 along y.
template <class T, int NDIM>
__device__ __forceinline__ void reg_face(const FaceRegEntry& e, const DevFlux<T>& F, T* __restrict__ reg, int nreg,
                                         int slot, T dt) {
  constexpr int ns = NDIM == 2 ? 6 : 5;
  constexpr int nmax = NDIM == 3 ? kR * kR : kR;
  const char* fd = F.base + (uint64_t)(7 * e.d) * F.stride;
  const char* fz = fd + (e.d == 0 ? 6 : 5) * F.stride;
  T v[nmax][ns];
#pragma unroll
  for (int i = 0; i < nmax; ++i) {
    if (i < e.n) {
#pragma unroll
      for (int q = 0; q < ns; ++q) v[i][q] = reinterpret_cast<const T*>(q < 5 ? fd + q * F.stride : fz)[e.e[i]];
    } else {
#pragma unroll
      for (int q = 0; q < ns; ++q) v[i][q] = T(0);
    }
  }
  T* out = reg + ((int64_t)slot * nreg + e.reg) * 6;
  const T inv = inv_count<T>(e.n);
#pragma unroll
  for (int q = 0; q < ns; ++q) {
    T m = T(0);
#pragma unroll
    for (int i = 0; i < nmax; ++i)
      if (i < e.n) m += v[i][q];
    int s = q;
    if (q >= 1 && q <= 3) {
      s = q + e.d;
      s = s > 3 ? s - 3 : s;
    }
    out[s] = dt * (m * inv);
  }
}

template <class T, bool UPWIND>
__device__ __forceinline__ void reg_edge(const EdgeRegEntry& e, const DevFlux<T>& F, T* __restrict__ reg, int nreg,
                                         int slot, T dt) {
  // faces of direction b = a + 1 (component 5) and c = a + 2 (component 6)
  const int b = e.a == 2 ? 0 : e.a + 1, c = e.a == 0 ? 2 : e.a - 1;
  const T* fb = reinterpret_cast<const T*>(F.base + (uint64_t)(7 * b + 5) * F.stride);
  const T* fc = reinterpret_cast<const T*>(F.base + (uint64_t)(7 * c + 6) * F.stride);
  const T* fe = UPWIND ? (e.a == 0 ? F.edge[0] : e.a == 1 ? F.edge[1] : F.edge[2]) : nullptr;
  T v[kR][4];
#pragma unroll
  for (int i = 0; i < kR; ++i) {
    v[i][0] = v[i][1] = v[i][2] = v[i][3] = T(0);
    if (i < e.n) {
      const int32_t x = e.e[i];
      if (UPWIND) {
        v[i][0] = fe[x];
      } else {
        v[i][0] = fb[x - e.st[1]];
        v[i][1] = fb[x];
        v[i][2] = fc[x - e.st[0]];
        v[i][3] = fc[x];
      }
    }
  }
  T m = T(0);
#pragma unroll
  for (int i = 0; i < kR; ++i)
    if (i < e.n) m += UPWIND ? v[i][0] : emf_mean(v[i][0], v[i][1], v[i][2], v[i][3]);
  reg[(int64_t)slot * nreg + e.reg] = dt * (m * inv_count<T>(e.n));
}

// The face and edge registers of every job of a launch cycle in one launch, a
// thread an entry.  What bounds it is the chain of dependent loads: the job,
// the entry, the fluxes.  A block lies in one job, so the job comes by scalar
// loads; the flux arrays are reached by their common base and stride instead
// of a pointer looked up by direction, and an edge's strides lie in its entry
// (a launch on 3 levels over 24^3 in FP64: 6.9 us, 11.4 before; over 64^2:
// 4.5 us, 8.1 before).
template <class T, int NDIM, bool UPWIND>
__global__ __launch_bounds__(kRegBlock) void k_registers(RegJobs<T> jobs, DevFlux<T> F,
                                                         const double* __restrict__ dt0p) {
  const double dt0 = dt0p[0];
  for (int blk = blockIdx.x; blk < jobs.blocks; blk += gridDim.x) {
    int j = 0;
#pragma unroll
    for (int k = 1; k < kMaxRegJobs; ++k) j += blk >= jobs.begin[k];
    const RegJob<T>& J = jobs.j[j];
    const T dt = T(dt0 / J.dt_div);
    const int i = (blk - jobs.begin[j]) * kRegBlock + (int)threadIdx.x;
    if (i < J.nf) reg_face<T, NDIM>(J.fe[i], F, J.freg, J.nfreg, J.slot, dt);
    else if (i < J.nf + J.ne) reg_edge<T, UPWIND>(J.ee[i - J.nf], F, J.ereg, J.nereg, J.slot, dt);
  }
}

// Reflux of one uncovered coarse cell.  Every load of a register's fields is
// issued before the first store of the cell's (one memory latency a register
// instead of one a field).
template <class T, int NDIM>
__device__ __forceinline__ void reflux_one(const RefluxEntry& e, const T* __restrict__ reg, int nreg,
                                           const DevState<T>& U) {
  constexpr int ns = NDIM == 2 ? 6 : 5;
  constexpr int imax = 6;
  T acc[ns];
#pragma unroll
  for (int q = 0; q < ns; ++q) acc[q] = U.f[q < 5 ? q : 7][e.cell];
#pragma unroll
  for (int i = 0; i < imax; ++i)
    if (i < e.n) {
      const T* r = reg + (int64_t)e.reg[i] * 6;
      T rc[ns], rf[ns][kR];
#pragma unroll
      for (int q = 0; q < ns; ++q) {
        rc[q] = r[q];
#pragma unroll
        for (int k = 0; k < kR; ++k) rf[q][k] = r[(int64_t)(k + 1) * nreg * 6 + q];
      }
#pragma unroll
      for (int q = 0; q < ns; ++q) {
        T fine = T(0);
#pragma unroll
        for (int k = 0; k < kR; ++k) fine += rf[q][k];
        const T delta = rc[q] - fine;
        acc[q] += T(e.coef[i]) * delta;
      }
    }
#pragma unroll
  for (int q = 0; q < ns; ++q) U.f[q < 5 ? q : 7][e.cell] = acc[q];
}

// EMF correction of one copy of an uncovered coarse face.
template <class T>
__device__ __forceinline__ void emffix_one(const EmfFixEntry& e, const T* __restrict__ reg, int nreg,
                                           const DevState<T>& U) {
  constexpr int imax = 4;
  {
    T rc[imax], rf[imax][kR];
#pragma unroll
    for (int i = 0; i < imax; ++i) {
      rc[i] = T(0);
#pragma unroll
      for (int k = 0; k < kR; ++k) rf[i][k] = T(0);
      if (i < e.n) {
        const T* r = reg + e.reg[i];
        rc[i] = r[0];
#pragma unroll
        for (int k = 0; k < kR; ++k) rf[i][k] = r[(int64_t)(k + 1) * nreg];
      }
    }
    T corr = T(0);
#pragma unroll
    for (int i = 0; i < imax; ++i)
      if (i < e.n) {
        T fine = T(0);
#pragma unroll
        for (int k = 0; k < kR; ++k) fine += rf[i][k];
        corr += T(e.coef[i]) * (fine - rc[i]);
      }
    U.f[5 + e.d][e.face] -= corr;
  }
}

// Restriction of one covered coarse cell or coarse face copy.
template <class T, int NDIM>
__device__ __forceinline__ void restrict_one(const RestrictEntry& e, const GridDesc* __restrict__ grids,
                                             const DevState<T>& Uf, const DevState<T>& Uc) {
  {
    const GridDesc G = grids[e.fgrid];
    const int64_t st[3] = {1, G.P[0], (int64_t)G.P[0] * G.P[1]};
    if (e.d < 0) {
      constexpr int ns = NDIM == 2 ? 6 : 5;
      constexpr int nz = NDIM == 3 ? kR : 1;
      T v[ns][nz * kR * kR];
#pragma unroll
      for (int q = 0; q < ns; ++q) {
        const int s = q < 5 ? q : 7;
#pragma unroll
        for (int kz = 0; kz < nz; ++kz)
#pragma unroll
          for (int ky = 0; ky < kR; ++ky)
#pragma unroll
            for (int kx = 0; kx < kR; ++kx)
              v[q][(kz * kR + ky) * kR + kx] = Uf.f[s][e.src + kx + ky * st[1] + kz * st[2]];
      }
#pragma unroll
      for (int q = 0; q < ns; ++q) {
        const int s = q < 5 ? q : 7;
        T m = T(0);
#pragma unroll
        for (int c = 0; c < nz * kR * kR; ++c) m += v[q][c];
        Uc.f[s][e.dst] = m / T(kR * kR * nz);
      }
    } else {
      const int d = e.d;
      const int a1 = (d + 1) % 3, a2 = (d + 2) % 3;
      const int n1 = a1 < NDIM ? kR : 1, n2 = a2 < NDIM ? kR : 1;
      T v[kR * kR];
#pragma unroll
      for (int i1 = 0; i1 < kR; ++i1)
#pragma unroll
        for (int i2 = 0; i2 < kR; ++i2)
          v[i1 * kR + i2] = (i1 < n1 && i2 < n2) ? Uf.f[5 + d][e.src + i1 * st[a1] + i2 * st[a2]] : T(0);
      T m = T(0);
#pragma unroll
      for (int i1 = 0; i1 < kR; ++i1)
#pragma unroll
        for (int i2 = 0; i2 < kR; ++i2)
          if (i1 < n1 && i2 < n2) m += v[i1 * kR + i2];
      Uc.f[5 + d][e.dst] = m / T(n1 * n2);
    }
  }
}

// One synchronisation in one launch: threads [0, nr) reflux uncovered
// coarse cells, the next ne correct uncovered coarse faces, the rest
// restrict covered cells and faces.  The three sets of outputs are disjoint
// and none reads another's outputs, so the order inside the launch is free.
template <class T, int NDIM>
__global__ __launch_bounds__(256) void k_sync(const RefluxEntry* __restrict__ rfx, int nr,
                                              const EmfFixEntry* __restrict__ efx, int ne,
                                              const RestrictEntry* __restrict__ rst, int nrs,
                                              const GridDesc* __restrict__ grids, const T* __restrict__ freg,
                                              int nfreg, const T* __restrict__ ereg, int nereg, DevState<T> Uf,
                                              DevState<T> Uc) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < nr + ne + nrs; t += gridDim.x * blockDim.x) {
    if (t < nr) reflux_one<T, NDIM>(rfx[t], freg, nfreg, Uc);
    else if (t < nr + ne) emffix_one<T>(efx[t - nr], ereg, nereg, Uc);
    else restrict_one<T, NDIM>(rst[t - nr - ne], grids, Uf, Uc);
  }
}

}  // namespace

template <class T>
void launch_register_jobs(int ndim, const RegJobs<T>& jobs, DevFlux<T> F, const double* dt0, bool upwind_emf,
                          hipStream_t s) {
  if (jobs.blocks <= 0) return;
  const dim3 grid(jobs.blocks < 65535 ? jobs.blocks : 65535), block(kRegBlock);
#define AMR_REGS(ND, U) hipLaunchKernelGGL((k_registers<T, ND, U>), grid, block, 0, s, jobs, F, dt0)
  if (ndim == 3) {
    if (upwind_emf) AMR_REGS(3, true);
    else AMR_REGS(3, false);
  } else {
    if (upwind_emf) AMR_REGS(2, true);
    else AMR_REGS(2, false);
  }
#undef AMR_REGS
}

template <class T>
void launch_sync(int ndim, int R, const GridDesc* grids, const SyncTables& t, const T* freg, const T* ereg,
                 DevState<T> Uf, DevState<T> Uc, hipStream_t s) {
  (void)R;  // the kernels are unrolled over kR; the caller checks R == kR
  const int n = t.n_reflux + t.n_emffix + t.n_restrict;
  if (n <= 0) return;
#define AMR_SYNC(ND)                                                                                              \
  hipLaunchKernelGGL((k_sync<T, ND>), dim3(blocks_for(n)), dim3(256), 0, s, t.d_reflux, t.n_reflux, t.d_emffix,   \
                     t.n_emffix, t.d_restrict, t.n_restrict, grids, freg, t.nfreg, ereg, t.nereg, Uf, Uc)
  if (ndim == 3) AMR_SYNC(3);
  else AMR_SYNC(2);
#undef AMR_SYNC
}

template void launch_register_jobs<float>(int, const RegJobs<float>&, DevFlux<float>, const double*, bool,
                                          hipStream_t);
template void launch_register_jobs<double>(int, const RegJobs<double>&, DevFlux<double>, const double*, bool,
                                           hipStream_t);
template void launch_sync<float>(int, int, const GridDesc*, const SyncTables&, const float*, const float*,
                                 DevState<float>, DevState<float>, hipStream_t);
template void launch_sync<double>(int, int, const GridDesc*, const SyncTables&, const double*, const double*,
                                  DevState<double>, DevState<double>, hipStream_t);

}  // namespace amr
