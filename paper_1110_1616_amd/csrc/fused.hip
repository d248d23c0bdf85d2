// Fused advance kernel for gfx950: the flux kernel's work (primitive
// recovery, minmod slopes, Hancock predictor, HLLD on every face) and the
// update kernel's work (edge EMFs, conservative and constrained-transport
// update) in one launch, so the face fluxes never travel through HBM.
//
// A work item is a column tile of tw x th threads over cells
// (x0-1+tx, y0-1+ty) marching along z.  Per plane k every active lane forms
// its cell's predicted face states; lanes then solve the Riemann problems of
// their cell's low x-face (tx >= 1), low y-face (ty >= 1) and low z-face
// (from the state carried from plane k-1), and the fluxes go to LDS, double
// buffered over two planes.  From them come the edge EMFs E_z of plane k and
// E_x, E_y at z = k - 1/2, and the update of plane k-1 (cells and their x-
// and y-faces) and of the z-faces at k - 1/2.  A plane takes two barriers in
// 3-D: the update reads E_z of the plane below (from the iteration before)
// and forms the neighbours' E_x, E_y again from their inputs in LDS.  A tile updates the cells of
// lanes tx in [1, tw-2], ty in [1, th-2] (their high faces and the edges
// around them are computed in the tile); tiles overlap by two columns and
// rows (the last x- and y-face of the update region go to the lane that
// holds them).  Every flux, EMF and update is formed with the same source
// expressions as the two-kernel path (the update's arithmetic is shared, in
// emf.hpp), and the library is compiled with multiply-add contraction
// inside single expressions only, so the results equal the two-kernel
// path's bit for bit.
//
// Face fluxes that the coarse/fine registers read afterwards are still
// stored: a per-element mask marks them (bit d for the face normal to d) and
// one owning lane per face writes them.
#include <algorithm>
#include <type_traits>

#include "advance_common.hpp"
#include "amr_internal.hpp"
#include "emf.hpp"
#include "launch_common.hpp"
#include "mhd_device.hpp"

namespace amr {

namespace {

// Both state sets, indexed by level parity per work item (a kernel-argument
// block read where an item starts, not held in registers across items).
template <class T> struct StatePair {
  DevState<T> s[2];
};
// A masked store of a face's seven flux components forms the arrays'
// addresses from the base and stride where it stores (the empty asm keeps
// the 21 addresses from being formed once and held in scalar registers
// through the plane loop, which spilled them).
template <class T, class B>
__device__ __forceinline__ void st_flux7(const DevFlux<T>& F, int d, B b, const T (&v)[7]) {
  uint64_t p = reinterpret_cast<uint64_t>(F.base), st = F.stride;
  asm volatile("" : "+s"(p), "+s"(st));
  p += (uint64_t)(7 * d) * st;
#pragma unroll
  for (int c = 0; c < 7; ++c) {
    *reinterpret_cast<__attribute__((address_space(1))) T*>(p + b) = v[c];
    p += st;
  }
}

// Lane t of a tile dimension tdim is the one that stores (for the
// registers) coordinate c of a computed range [clo, chi]: tiles overlap by
// two, so interior lanes [1, tdim-2] own their coordinate and the edge lanes
// only the range's end points.
__device__ __forceinline__ bool owns(int t, int tdim, int c, int clo, int chi) {
  return (t >= 1 && t <= tdim - 2) || (t == 0 && c == clo) || (t == tdim - 1 && c == chi);
}

template <class T, int NDIM, bool PERSIST>
__global__ __launch_bounds__(256) void k_fused(const GridDesc* __restrict__ grids, const FluxItem* __restrict__ items,
                                               int nitems, StatePair<T> S, uint32_t parity,
                                               DevFlux<T> F, const uint8_t* __restrict__ fmask,
                                               const double* __restrict__ dt0p, Phys ph, ErrBlock* err, WorkQueue* q,
                                               bool xcd, int claim) {
  __shared__ T sW[8][kMaxPlane + 1];  // (the last entry takes the writes of lanes outside the tile)
  __shared__ T sX[7][256];
  __shared__ T sY[7][256];
  __shared__ T sH[2][10][256];  // hydro components 0..4 of the x- (0..4) and y-face (5..9) fluxes, by plane parity
  __shared__ T sB[4][256];      // EMF inputs of this plane: F_x c5, F_y c6, F_z c5, F_z c6 (2-D: F_x c6, F_y c5)
  __shared__ T sEz[2][256];     // E_z at each lane's (x, y) low corner, by plane parity
  __shared__ T sX6[2][256];     // 3-D: F_x c6 and F_y c5 of each lane, by plane parity (the inputs of
  __shared__ T sY5[2][256];     // the neighbours' E_x, E_y, formed again where the z-faces need them)
  __shared__ int s_claim[2], s_c;
  if (threadIdx.x == 0) s_c = 0;

  const int tid = threadIdx.x;
  const T gam = T(ph.gamma);
  const T gm1 = gam - T(1);
  const T gm1_inv = drcp(gm1);

  ItemRange rng = first_claim<PERSIST>(nitems, claim, xcd);
  for (;;) {
    const int it = next_item<PERSIST>(rng, nitems, claim, q, s_claim, &s_c, xcd);
    if (it < 0) break;
    const FluxItem item = items[it];
    const GridDesc G = grids[item.grid];
    const bool odd = (parity >> G.level) & 1u;
    const DevState<T> U = S.s[odd ? 1 : 0];
    const DevState<T> V = S.s[odd ? 0 : 1];
    const Idx<NDIM> ix(G);
    const IdxB<NDIM, T> bx(G);
    const int gv = item.gv;
    const int cl = -gv + 1;
    const int chx = G.n[0] + gv - 1, chy = G.n[1] + gv - 1;
    const int wlo = -gv, whix = G.n[0] + gv, whiy = G.n[1] + gv;
    const int ul = -gv + 2;
    const int uhx = G.n[0] + gv - 2, uhy = G.n[1] + gv - 2, uhz = NDIM == 3 ? G.n[2] + gv - 2 : 1;
    const int x0 = item.x0, y0 = item.y0;
    const int tw = item.tw, th = 256 / tw, kW = tw + 2;
    const int tx = tid % tw, ty = tid / tw;
    const bool live = ty < th;
    const int cx = x0 - 1 + tx, cy = y0 - 1 + ty;
    const bool act = live && cx >= cl && cx < chx && cy >= cl && cy < chy;
    const bool xf = act && tx >= 1 && cx > cl;  // its cell's low x-face is a face of the launch
    const bool yf = act && ty >= 1 && cy > cl;  // low y-face
    // update ownership: cells and z-faces at interior lanes; x- and y-faces
    // also the update region's last face (uh), wherever it falls
    const bool ucol = tx >= 1 && tx <= tw - 2 && cx >= ul && cx < uhx;
    const bool urow = ty >= 1 && ty <= th - 2 && cy >= ul && cy < uhy;
    const bool ucell = live && ucol && urow;
    const bool ubx = live && urow && (ucol || (tx >= 1 && cx == uhx));
    const bool uby = live && ucol && (urow || (ty >= 1 && cy == uhy));
    // flux stores for the registers: one owning lane per computed face (mask
    // bits of the faces this lane stores)
    const bool sxy = owns(tx, tw, cx, cl, chx - 1) && owns(ty, th, cy, cl, chy - 1);
    const unsigned smask = sxy ? (xf ? 1u : 0u) | (yf ? 2u : 0u) | (act ? 4u : 0u) : 0u;
    // Every lane runs the whole plane: lanes without a cell of the launch
    // load a clamped cell of the box and read clamped LDS entries, and what
    // they form is used by nobody (a lone wave of a SIMD issues one
    // instruction every four cycles, scalar or vector, so execution masks
    // around each piece cost more than the idle lanes).
    const int lx = min(max(cx, wlo), whix - 1), ly = min(max(cy, wlo), whiy - 1);
    const int tl = max(tid - 1, 0), td = max(tid - tw, 0);        // low x and y neighbours
    const int tr = min(tid + 1, 255), tu = min(tid + tw, 255);    // high ones

    double rl = 1.0;
    for (int l = 0; l < G.level; ++l) rl *= (double)ph.ratio;
    const T dt = T(dt0p[0] / rl);
    const T cdx = dt * T(rl / ph.dx0[0]), cdy = dt * T(rl / ph.dx0[1]);
    const T cdz = dt * T(NDIM == 3 ? rl / ph.dx0[2] : 0.0);

    const int eo = live ? (ty + 1) * kW + tx + 1 : kW + 1;  // LDS plane entry read around
    const int ew = live ? eo : kMaxPlane;                   // and written
    const int nring = 2 * (tw + th);
    int rex = 0, rey = 0;
    if (tid < nring) ring_entry(tid, tw, th, rex, rey);
    const int rcx = x0 - 2 + rex, rcy = y0 - 2 + rey;
    const bool ring = tid < nring;
    const bool rok = ring && rcx >= wlo && rcx < whix && rcy >= wlo && rcy < whiy;

    // planes: update planes [z0, z1) (cells below uhz; z-faces up to uhz);
    // predicted states from z0 - 1 to the last plane whose fluxes they need
    const int z0 = NDIM == 3 ? item.z0 : 0, z1 = NDIM == 3 ? item.z1 : 1;
    const int kstart = NDIM == 3 ? z0 - 1 : 0;
    const int kend = NDIM == 3 ? min(z1, uhz) : 0;  // inclusive

    T dzm[8], wcur[8], wnext[8], wring[8];  // dzm: wcur minus the plane below
    T fbcur[3][2], fbnext[3][2];
    T zcarry[7];
#pragma unroll
    for (int c = 0; c < 8; ++c) { dzm[c] = T(0); wnext[c] = T(1); wring[c] = T(1); }
#pragma unroll
    for (int c = 0; c < 7; ++c) zcarry[c] = T(1);
    // carried from the previous plane: z-flux hydro components at k - 1/2,
    // E_x and E_y at the low z-edges, F_y c5 and F_x c6 of the plane
    T fzp[5] = {T(0), T(0), T(0), T(0), T(0)};
    T exp_ = T(0), eyp_ = T(0), fy5p = T(0), fx6p = T(0);

#pragma unroll
    for (int d = 0; d < 3; ++d) fbcur[d][0] = fbcur[d][1] = fbnext[d][0] = fbnext[d][1] = T(0);
    if (NDIM == 3) {
      // the item's first planes: every load issued before any conversion
      T r0[5], r1[5], r2[5], rr[5], f0[3][2], fr[3][2], wprev[8];
      load_raw3<T>(U, bx(lx, ly, kstart - 1), bx.sy, bx.sz, r0, f0);
      load_raw3<T>(U, bx(lx, ly, kstart), bx.sy, bx.sz, r1, fbcur);
      load_raw3<T>(U, bx(lx, ly, kstart + 1), bx.sy, bx.sz, r2, fbnext);
      if (rok) load_raw3<T>(U, bx(rcx, rcy, kstart), bx.sy, bx.sz, rr, fr);
      raw3_to_prim<T>(r0, f0, gm1, wprev);
      raw3_to_prim<T>(r1, fbcur, gm1, wcur);
      raw3_to_prim<T>(r2, fbnext, gm1, wnext);
      if (rok) raw3_to_prim<T>(rr, fr, gm1, wring);
#pragma unroll
      for (int c = 0; c < 8; ++c) dzm[c] = wcur[c] - wprev[c];
    } else {
      load_prim_faces_b<T, NDIM>(U, bx(lx, ly, kstart), bx.sy, bx.sz, gm1, wcur, fbcur);
      if (rok) load_prim_b<T, NDIM>(U, bx(rcx, rcy, kstart), bx.sy, bx.sz, gm1, wring);
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      sW[c][ew] = wcur[c];
      if (ring) sW[c][rey * kW + rex] = wring[c];
    }
    __syncthreads();

    unsigned mknext = fmask ? fmask[ix(lx, ly, kstart)] : 0u;
    for (int k = kstart; k <= kend; ++k) {
      const int pb = k & 1;
      // this plane's face mask was loaded an iteration ago; the next one's
      // load is in flight through this iteration
      const unsigned mk = mknext & smask;
      if (fmask && k + 1 <= kend) mknext = fmask[ix(lx, ly, k + 1)];
      T rnext[5], rfb[3][2], rring[5], rrfb[3][2];
      const bool rn = NDIM == 3 && rok && k + 1 <= kend;
      if (NDIM == 3) {
        // (the last iterations load the last plane again: no branch)
        load_raw3<T>(U, bx(lx, ly, min(k + 2, kend + 1)), bx.sy, bx.sz, rnext, rfb);
        if (rn) load_raw3<T>(U, bx(rcx, rcy, k + 1), bx.sy, bx.sz, rring, rrfb);
      }
      Pred<T, NDIM> pr;
      T dzp[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) dzp[c] = wnext[c] - wcur[c];
      {
        T wxm[8], wxp[8], wym[8], wyp[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          wxm[c] = sW[c][eo - 1];
          wxp[c] = sW[c][eo + 1];
          wym[c] = sW[c][eo - kW];
          wyp[c] = sW[c][eo + kW];
        }
        const T hcdt[3] = {T(0.5) * cdx, T(0.5) * cdy, T(0.5) * cdz};
        const bool ok = predict<T, NDIM>(wcur, wxm, wxp, wym, wyp, dzm, dzp, fbcur, hcdt, gm1, gm1_inv, pr);
        if (act && (!ok || wcur[0] <= T(0) || wcur[4] <= T(0))) flag_bad(err, ix(cx, cy, k));
#pragma unroll
        for (int c = 0; c < 7; ++c) {
          sX[c][tid] = pr.p[0][c];
          sY[c][tid] = pr.p[1][c];
        }
      }
      __syncthreads();
      // this plane's W has been read: the next plane's goes into LDS while
      // the Riemann problems run
      T bn[3] = {fbcur[0][0], fbcur[1][0], fbcur[2][0]};
      if (NDIM == 3) {
        if (rn) raw3_to_prim<T>(rring, rrfb, gm1, wring);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          sW[c][ew] = wnext[c];
          if (ring) sW[c][rey * kW + rex] = wring[c];
          dzm[c] = dzp[c];
          wcur[c] = wnext[c];
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          fbcur[d][0] = fbnext[d][0];
          fbcur[d][1] = fbnext[d][1];
        }
        raw3_to_prim<T>(rnext, rfb, gm1, wnext);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          fbnext[d][0] = rfb[d][0];
          fbnext[d][1] = rfb[d][1];
        }
      }
      const bool zf = NDIM == 3 && k >= z0;
      const auto eb = bx(lx, ly, k);
      T fx[7], fy[7], fz[7];
#pragma unroll
      for (int c = 0; c < 7; ++c) fz[c] = T(0);
      {
        T l[7];
#pragma unroll
        for (int c = 0; c < 7; ++c) l[c] = sX[c][tl];
        hlld7(l, pr.m[0], bn[0], gam, gm1_inv, fx);
      }
      {
        T l[7];
#pragma unroll
        for (int c = 0; c < 7; ++c) l[c] = sY[c][td];
        hlld7(l, pr.m[1], bn[1], gam, gm1_inv, fy);
      }
      if (zf) hlld7(zcarry, pr.m[2], bn[2], gam, gm1_inv, fz);
      if (mk != 0u) {
        const bool own = NDIM == 2 || (k >= z0 && k < z1);
        if ((mk & 1u) && (own || (k == kstart && z0 == ul))) st_flux7(F, 0, eb, fx);
        if ((mk & 2u) && (own || (k == kstart && z0 == ul))) st_flux7(F, 1, eb, fy);
        if (NDIM == 3 && (mk & 4u) && own) st_flux7(F, 2, eb, fz);
      }
      if (NDIM == 3) {
#pragma unroll
        for (int c = 0; c < 7; ++c) zcarry[c] = pr.p[2][c];
      }
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        sH[pb][c][tid] = fx[c];
        sH[pb][5 + c][tid] = fy[c];
      }
      sB[0][tid] = fx[5];
      sB[1][tid] = fy[6];
      if (NDIM == 3) {
        sB[2][tid] = fz[5];
        sB[3][tid] = fz[6];
        sX6[pb][tid] = fx[6];
        sY5[pb][tid] = fy[5];
      } else {
        sB[2][tid] = fx[6];
        sB[3][tid] = fy[5];
      }
      __syncthreads();
      // edge EMFs: E_z at (cx - 1/2, cy - 1/2) of plane k; E_x at
      // (cx, cy - 1/2) and E_y at (cx - 1/2, cy), both at z = k - 1/2
      sEz[pb][tid] = emf_mean(sB[0][td], fx[5], sB[1][tl], fy[6]);
      // 2-D: the faces read E_z of the neighbours' corners, formed above; in
      // 3-D every input of this plane's update is in LDS already (E_z of the
      // plane below, and the inputs of the neighbours' E_x, E_y)
      if (NDIM == 2) __syncthreads();
      if (NDIM == 3) {
        const T ex = emf_mean(fy5p, fy[5], sB[3][td], fz[6]);
        const T ey = emf_mean(sB[2][tl], fz[5], fx6p, fx[6]);
        // the old values of everything this plane updates are loaded before
        // any store, so their latencies overlap
        const int kk = k - 1;
        const bool zup = ucell && k >= z0 && k < z1;
        const bool cup = kk >= z0 && kk < z1 && kk < uhz;
        const auto ec = bx(lx, ly, kk);
        T uo[8];
        uo[7] = ldb(U.f[7], eb);
#pragma unroll
        for (int s = 0; s < 7; ++s) uo[s] = ldb(U.f[s], ec);
        // z-faces at k - 1/2 (element of plane k): E_y of the next lane's and
        // E_x of the next row's low z-edge, from the same inputs as those
        // lanes form them
        const int qb = kk & 1;
        const T ey1 = emf_mean(sB[2][tid], sB[2][tr], sX6[qb][tr], sX6[pb][tr]);
        const T ex1 = emf_mean(sY5[qb][tu], sY5[pb][tu], sB[3][tid], sB[3][tu]);
        if (zup) stb(V.f[7], eb, uo[7] - curl_delta(cdx, ey1, ey, cdy, ex1, ex));
        // cells and x-, y-faces of plane k - 1
        if (cup) {
          const T ez0 = sEz[qb][tid], ezy = sEz[qb][tu], ezx = sEz[qb][tr];
          T un[5];
#pragma unroll
          for (int s = 0; s < 5; ++s) {
            const int qx = hydro_comp(s, 0), qy = hydro_comp(s, 1), qz = hydro_comp(s, 2);
            const T acc = flux_delta<T, 3>(cdx, sH[qb][qx][tr], sH[qb][qx][tid], cdy, sH[qb][5 + qy][tu],
                                           sH[qb][5 + qy][tid], cdz, fz[qz], fzp[qz]);
            un[s] = uo[s] - acc;
          }
          if (ucell)
#pragma unroll
            for (int s = 0; s < 5; ++s) stb(V.f[s], ec, un[s]);
          if (ubx) stb(V.f[5], ec, uo[5] - curl_delta(cdy, ezy, ez0, cdz, ey, eyp_));
          if (uby) stb(V.f[6], ec, uo[6] - curl_delta(cdz, ex, exp_, cdx, ezx, ez0));
        }
#pragma unroll
        for (int c = 0; c < 5; ++c) fzp[c] = fz[c];
        exp_ = ex;
        eyp_ = ey;
        fy5p = fy[5];
        fx6p = fx[6];
      } else {
        // 2-D: the single plane's cells (B_z cell-centred) and faces
        T uo[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) uo[s] = ldb(U.f[s], eb);
        if (ucell) {
#pragma unroll
          for (int s = 0; s < 5; ++s) {
            const int qx = hydro_comp(s, 0), qy = hydro_comp(s, 1);
            const T acc = flux_delta<T, 2>(cdx, sH[0][qx][tr], sH[0][qx][tid], cdy, sH[0][5 + qy][tu],
                                           sH[0][5 + qy][tid], T(0), T(0), T(0));
            stb(V.f[s], eb, uo[s] - acc);
          }
          const T acc = flux_delta<T, 2>(cdx, sB[2][tr], sB[2][tid], cdy, sB[3][tu], sB[3][tid], T(0), T(0), T(0));
          stb(V.f[7], eb, uo[7] - acc);
        }
        if (ubx) stb(V.f[5], eb, uo[5] - face_delta2(cdy, sEz[0][tu], sEz[0][tid]));
        if (uby) stb(V.f[6], eb, uo[6] + face_delta2(cdx, sEz[0][tr], sEz[0][tid]));
      }
    }
    __syncthreads();
  }
  retire<PERSIST>(q);
}

}  // namespace

template <class T>
void launch_fused(int ndim, const GridDesc* grids, const FluxItem* items, int nitems, DevState<T> S0, DevState<T> S1,
                  uint32_t parity, DevFlux<T> F, const uint8_t* fmask, const double* dt0, Phys ph, ErrBlock* err,
                  WorkQueue* q, int pblocks, bool xcd, int claim, hipStream_t s) {
  if (nitems <= 0) return;
  const bool per = pblocks > 0 && q != nullptr;
  const dim3 grid(per ? std::min(pblocks, nitems) : claim_blocks(nitems, claim, xcd)), block(256);
  StatePair<T> SP;
  SP.s[0] = S0;
  SP.s[1] = S1;
#define AMR_FUSED_LAUNCH(ND, P) \
  hipLaunchKernelGGL((k_fused<T, ND, P>), grid, block, 0, s, grids, items, nitems, SP, parity, F, fmask, dt0, ph, err, q, \
                     xcd, claim)
  if (ndim == 3) {
    if (per) AMR_FUSED_LAUNCH(3, true);
    else AMR_FUSED_LAUNCH(3, false);
  } else {
    if (per) AMR_FUSED_LAUNCH(2, true);
    else AMR_FUSED_LAUNCH(2, false);
  }
#undef AMR_FUSED_LAUNCH
}

template <class T> int fused_occupancy(int ndim) {
  int a = 0;
  if (ndim == 3)
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, k_fused<T, 3, true>, 256, 0);
  else
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, k_fused<T, 2, true>, 256, 0);
  return a > 0 ? a : 1;
}

#define AMR_FUSED_INST(T)                                                                                           \
  template void launch_fused<T>(int, const GridDesc*, const FluxItem*, int, DevState<T>, DevState<T>, uint32_t,    \
                                DevFlux<T>, const uint8_t*, const double*, Phys, ErrBlock*, WorkQueue*, int, bool, \
                                int, hipStream_t);                                                                      \
  template int fused_occupancy<T>(int);
AMR_FUSED_INST(float)
AMR_FUSED_INST(double)
#undef AMR_FUSED_INST

}  // namespace amr
