// Fused advance kernel for gfx950: the flux kernel's work (primitive
// recovery, minmod slopes, Hancock predictor, HLLD on every face) and the
// update kernel's work (edge EMFs, conservative and constrained-transport
// update) in one launch, so the face fluxes never travel through HBM.
//
// A work item is a column tile of tw x th threads over cells
// (x0-1+tx, y0-1+ty) marching along z.  Per plane k every lane forms its
// cell's predicted face states and solves the Riemann problems of the cell's
// low x-, y- and z-face (the z one from the state carried from plane k-1);
// the fluxes go to LDS, where the face states were, and from them come the
// edge EMFs E_z of plane k and E_x, E_y at z = k - 1/2 of the lane and of its
// neighbours, the update of plane k-1 (cells and their x- and y-faces) and
// of the z-faces at k - 1/2.  What plane k's update needs of its own fluxes
// is carried as two values a field.  A tile updates the cells of
// lanes tx in [1, tw-2], ty in [1, th-2] (their high faces and the edges
// around them are computed in the tile); tiles overlap by two columns and
// rows (the last x- and y-face of the update region go to the lane that
// holds them).  Every flux, EMF and update is formed with the same source
// expressions as the two-kernel path (the update's arithmetic is shared, in
// emf.hpp), and the library is compiled with multiply-add contraction
// inside single expressions only, so the results equal the two-kernel
// path's bit for bit.
//
// What bounds it: instruction issue.  A plane takes about 1860 vector and
// 450 other instructions a wave in FP64; a wave alone on its SIMD issues at
// most one of any kind every four cycles and waits for LDS, barriers and
// dependent FP64 results in between, so two waves share each SIMD: 256
// registers (a dozen values in scratch) and 81 KB of LDS a block in FP64, two
// blocks a CU (157 registers in FP32, three).  To fit, the z differences wait in LDS, W of the next
// plane is read back from the W plane, and the loads of the next planes are
// issued behind the Riemann problems instead of a plane ahead.  Against one
// block a CU with 375 registers, 115 KB and the loads a plane ahead: two
// steps of a 128^3 grid 770 -> 628 us, two coarse steps of the 549-grid
// hierarchy 6225 -> 5442 us (FP32: the same within 1%); 654 and 5450 us since
// the fast speeds are divided by the density and both z-fluxes are carried.  Four waves a SIMD
// in FP32 (128 registers) spill and are 11% slower.  Waves in two roles, one
// predicting plane k + 1 while another solves plane k, pass every face state
// through LDS and were 12% slower (14% on the hierarchy).
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

// 2-D: the tile is one plane.
template <class T, bool PERSIST>
__global__ __launch_bounds__(256) void k_fused2(const GridDesc* __restrict__ grids, const FluxItem* __restrict__ items,
                                                int nitems, StatePair<T> S, uint32_t parity, DevFlux<T> F,
                                                const uint8_t* __restrict__ fmask, const double* __restrict__ dt0p,
                                                Phys ph, ErrBlock* err, WorkQueue* q, bool xcd, int claim) {
  constexpr int NDIM = 2;
  __shared__ T sW[8][kMaxPlane + 1];  // (the last entry takes the writes of lanes outside the tile)
  // the plane's high face states (x in 0..6, y in 7..13), then its fluxes
  __shared__ T sF[14][256];
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
    const int uhx = G.n[0] + gv - 2, uhy = G.n[1] + gv - 2;
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
    // they form is used by nobody (masks around each piece cost scalar
    // instructions, which share the waves' issue slots).
    const int lx = min(max(cx, wlo), whix - 1), ly = min(max(cy, wlo), whiy - 1);
    const int tl = max(tid - 1, 0), td = max(tid - tw, 0);        // low x and y neighbours
    const int tr = min(tid + 1, 255), tu = min(tid + tw, 255);    // high ones
    const int tdr = max(tid - tw + 1, 0), tul = min(tid + tw - 1, 255);  // low y of the high x, and the reverse

    double rl = 1.0;
    for (int l = 0; l < G.level; ++l) rl *= (double)ph.ratio;
    const T dt = T(dt0p[0] / rl);
    const T cdx = dt * T(rl / ph.dx0[0]), cdy = dt * T(rl / ph.dx0[1]);

    const int eo = live ? (ty + 1) * kW + tx + 1 : kW + 1;  // LDS plane entry read around
    const int ew = live ? eo : kMaxPlane;                   // and written
    const int nring = 2 * (tw + th);
    int rex = 0, rey = 0;
    if (tid < nring) ring_entry(tid, tw, th, rex, rey);
    const int rcx = x0 - 2 + rex, rcy = y0 - 2 + rey;
    const bool ring = tid < nring;
    const bool rok = ring && rcx >= wlo && rcx < whix && rcy >= wlo && rcy < whiy;

    T w[8], fb[3][2];
    {
      T wring[8];
      load_prim_faces_b<T, NDIM>(U, bx(lx, ly, 0), bx.sy, bx.sz, gm1, w, fb);
      if (rok) load_prim_b<T, NDIM>(U, bx(rcx, rcy, 0), bx.sy, bx.sz, gm1, wring);
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        sW[c][ew] = w[c];
        if (ring) sW[c][rey * kW + rex] = rok ? wring[c] : T(1);
      }
    }
    const unsigned mk = (fmask ? fmask[ix(lx, ly, 0)] : 0u) & smask;
    const auto eb = bx(lx, ly, 0);
    T uo[8];  // the old values of everything the tile updates
#pragma unroll
    for (int s = 0; s < 8; ++s) uo[s] = ldb(U.f[s], eb);
    __syncthreads();
    T ml[2][7];
    {
      T wxm[8], wxp[8], wym[8], wyp[8], sl[3][8], du[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        wxm[c] = sW[c][eo - 1];
        wxp[c] = sW[c][eo + 1];
        wym[c] = sW[c][eo - kW];
        wyp[c] = sW[c][eo + kW];
      }
      const T hcdt[3] = {T(0.5) * cdx, T(0.5) * cdy, T(0)};
      hancock_slopes<T, NDIM>(w, wxm, wxp, wym, wyp, w, w, fb, hcdt, gm1_inv, sl, du);
      const bool ok = hancock_states<T, NDIM>(w, sl, du, fb, gm1, gm1_inv,
                                              [&](int d, const T (&lo)[7], const T (&hi)[7]) {
#pragma unroll
                                                for (int c = 0; c < 7; ++c) {
                                                  ml[d][c] = lo[c];
                                                  sF[7 * d + c][tid] = hi[c];
                                                }
                                              });
      if (act && (!ok || w[0] <= T(0) || w[4] <= T(0))) flag_bad(err, ix(cx, cy, 0));
    }
    __syncthreads();
    T fx[7], fy[7], l[7];
#pragma unroll
    for (int c = 0; c < 7; ++c) l[c] = sF[c][tl];
    hlld7(l, ml[0], fb[0][0], gam, gm1_inv, fx);
#pragma unroll
    for (int c = 0; c < 7; ++c) l[c] = sF[7 + c][td];
    hlld7(l, ml[1], fb[1][0], gam, gm1_inv, fy);
    __syncthreads();  // the face states have been read: the fluxes take their place
#pragma unroll
    for (int c = 0; c < 7; ++c) {
      sF[c][tid] = fx[c];
      sF[7 + c][tid] = fy[c];
    }
    if (mk & 1u) st_flux7(F, 0, eb, fx);
    if (mk & 2u) st_flux7(F, 1, eb, fy);
    __syncthreads();
    // E_z at this lane's (cx - 1/2, cy - 1/2) corner and at its high x and
    // high y neighbours', from the inputs those lanes form theirs from
    const T ez0 = emf_mean(sF[5][td], fx[5], sF[13][tl], fy[6]);
    const T ezx = emf_mean(sF[5][tdr], sF[5][tr], fy[6], sF[13][tr]);
    const T ezy = emf_mean(fx[5], sF[5][tu], sF[13][tul], sF[13][tu]);
    if (ucell) {
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        const int qx = hydro_comp(s, 0), qy = hydro_comp(s, 1);
        stb(V.f[s], eb, uo[s] - flux_delta2<T>(cdx, sF[qx][tr], fx[qx], cdy, sF[7 + qy][tu], fy[qy]));
      }
      stb(V.f[7], eb, uo[7] - flux_delta2<T>(cdx, sF[6][tr], fx[6], cdy, sF[12][tu], fy[5]));
    }
    if (ubx) stb(V.f[5], eb, uo[5] - face_delta2(cdy, ezy, ez0));
    if (uby) stb(V.f[6], eb, uo[6] + face_delta2(cdx, ezx, ez0));
    __syncthreads();
  }
  retire<PERSIST>(q);
}

// 3-D: the tile marches along z.  Two blocks share a CU.
template <class T, bool PERSIST>
__global__ __launch_bounds__(256, (sizeof(T) == 8 ? 2 : 3)) void k_fused3(
    const GridDesc* __restrict__ grids, const FluxItem* __restrict__ items, int nitems, StatePair<T> S,
    uint32_t parity, DevFlux<T> F, const uint8_t* __restrict__ fmask, const double* __restrict__ dt0p, Phys ph,
    ErrBlock* err, WorkQueue* q, bool xcd, int claim) {
  constexpr int NDIM = 3;
  __shared__ T sW[8][kMaxPlane + 1];  // W of a plane (the last entry takes the writes of lanes outside the tile)
  // one plane's high face states (x in 0..6, y in 7..13), then its fluxes:
  // F_x in 0..6, F_y in 7..13, the two EMF components of F_z in 14, 15
  __shared__ T sF[16][256];
  __shared__ T sD[8][256];  // W of the lane's cell minus the plane below
  // What the update of the plane below needs next to `up` and fits no registers
  // in FP64: F_x c6 and F_y c5 of its lanes and the lane's F_z of the density.
  constexpr bool kPark = sizeof(T) == 8;
  __shared__ T sP[kPark ? 3 : 1][kPark ? 256 : 1];
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
    const int uhx = G.n[0] + gv - 2, uhy = G.n[1] + gv - 2;
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
    // they form is used by nobody (masks around each piece cost scalar
    // instructions, which share the waves' issue slots).
    const int lx = min(max(cx, wlo), whix - 1), ly = min(max(cy, wlo), whiy - 1);
    const int tl = max(tid - 1, 0), td = max(tid - tw, 0);        // low x and y neighbours
    const int tr = min(tid + 1, 255), tu = min(tid + tw, 255);    // high ones
    const int tdr = max(tid - tw + 1, 0), tul = min(tid + tw - 1, 255);  // low y of the high x, and the reverse

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
    const int uhz = G.n[2] + gv - 2;
    const int z0 = item.z0, z1 = item.z1;
    const int kstart = z0 - 1;
    const int kend = min(z1, uhz);  // inclusive

    const bool rwave = __builtin_amdgcn_readfirstlane(tid) < nring;  // (waves without ring lanes skip the ring)
    const int rx = rok ? rcx : lx, ry = rok ? rcy : ly, rw = rok ? rey * kW + rex : kMaxPlane;

    T wnext[8], fb[3][2], zlo[7];  // W of plane k + 1; face fields of plane k; high z states of plane k - 1
#pragma unroll
    for (int c = 0; c < 7; ++c) zlo[c] = T(1);
    // carried from the plane below: the terms of the x- and y-faces in the
    // updates of its cells, those of the E_z in its x- and y-faces', what the
    // z-faces' and E_x, E_y above it are subtracted from (the hydro F_z, ey and
    // ex), and the EMF inputs F_y c5, F_x c6 of the lane, of its high x (F_x c6)
    // and high y (F_y c5).  (With the z terms' low parts subtracted at once it is
    // one value a field and 128^3 takes 652 instead of 666 us, but c F_low and
    // c F_high rounded apart do not cancel where they are equal: 3000 times the
    // error in m_z of 1e-5 next to a pressure of 1 that does not depend on z.)
    T up[7] = {T(0), T(0), T(0), T(0), T(0), T(0), T(0)};
    T zl[7] = {T(0), T(0), T(0), T(0), T(0), T(0), T(0)};
    T fy5p = T(0), fx6p = T(0), fx6r = T(0), fy5u = T(0);
    {
      // the item's first planes: every load issued before any conversion
      T r0[5], r1[5], r2[5], rr[5], f0[3][2], f2[3][2], fr[3][2], w0[8], w1[8], wring[8];
      load_raw3<T>(U, bx(lx, ly, kstart - 1), bx.sy, bx.sz, r0, f0);
      load_raw3<T>(U, bx(lx, ly, kstart), bx.sy, bx.sz, r1, fb);
      load_raw3<T>(U, bx(lx, ly, kstart + 1), bx.sy, bx.sz, r2, f2);
      load_raw3<T>(U, bx(rx, ry, kstart), bx.sy, bx.sz, rr, fr);
      raw3_to_prim<T>(r0, f0, gm1, w0);
      raw3_to_prim<T>(r1, fb, gm1, w1);
      raw3_to_prim<T>(r2, f2, gm1, wnext);
      raw3_to_prim<T>(rr, fr, gm1, wring);
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        sD[c][tid] = w1[c] - w0[c];
        if (kPark && c < 3) sP[c][tid] = T(0);
        if (ring && !rok) sW[c][rey * kW + rex] = T(1);
        sW[c][rw] = wring[c];
        sW[c][ew] = w1[c];
      }
    }
    unsigned mk = (fmask ? ldb(fmask, bx(lx, ly, kstart) / (unsigned)sizeof(T)) : 0u) & smask;
    __syncthreads();
    for (int k = kstart; k <= kend; ++k) {
      T ml[3][7], zhi[7];  // low face states; the high z state
      {
        T w[8], sl[3][8], du[8];
        {
          T wxm[8], wxp[8], wym[8], wyp[8], dzm[8], dzp[8];
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            w[c] = sW[c][eo];
            dzm[c] = sD[c][tid];
            dzp[c] = wnext[c] - w[c];
            sD[c][tid] = dzp[c];
            wxm[c] = sW[c][eo - 1];
            wxp[c] = sW[c][eo + 1];
            wym[c] = sW[c][eo - kW];
            wyp[c] = sW[c][eo + kW];
          }
          const T hcdt[3] = {T(0.5) * cdx, T(0.5) * cdy, T(0.5) * cdz};
          hancock_slopes<T, NDIM>(w, wxm, wxp, wym, wyp, dzm, dzp, fb, hcdt, gm1_inv, sl, du);
#pragma unroll
          for (int d = 0; d < 3; ++d) form_now(sl[d]);
          form_now(du);
        }
        __syncthreads();  // the plane below's fluxes have been read: the face states take their place
        if constexpr (kPark) {  // (two free arrays until this plane's F_z)
          sF[14][tid] = zl[1];
          sF[15][tid] = zl[2];
        }
        const bool ok = hancock_states<T, NDIM>(w, sl, du, fb, gm1, gm1_inv,
                                                [&](int d, const T (&lo)[7], const T (&hi)[7]) {
#pragma unroll
                                                  for (int c = 0; c < 7; ++c) {
                                                    ml[d][c] = lo[c];
                                                    if (d == 2) zhi[c] = hi[c];
                                                    else sF[7 * d + c][tid] = hi[c];
                                                  }
                                                });
        if (act && (!ok || w[0] <= T(0) || w[4] <= T(0))) flag_bad(err, ix(cx, cy, k));
      }
      const T bn[3] = {fb[0][0], fb[1][0], fb[2][0]};
#pragma unroll
      for (int d = 0; d < 3; ++d) form_now(ml[d]);
      form_now(zhi);
      __syncthreads();  // this plane's W has been read, the face states are in place
#pragma unroll
      for (int c = 0; c < 8; ++c) sW[c][ew] = wnext[c];
      const auto eb = bx(lx, ly, k), ep = bx(lx, ly, k - 1), en = bx(lx, ly, min(k + 1, kend + 1));
      const bool own = (k >= z0 && k < z1) || (k == kstart && z0 == ul);
      T fx[7], fy[7], fz[7];
      {
        T l7[7];
#pragma unroll
        for (int c = 0; c < 7; ++c) l7[c] = sF[c][tl];
        hlld7(l7, ml[0], bn[0], gam, gm1_inv, fx);
      }
      {
        T l7[7];
#pragma unroll
        for (int c = 0; c < 7; ++c) l7[c] = sF[7 + c][td];
        hlld7(l7, ml[1], bn[1], gam, gm1_inv, fy);
      }
      // the loads behind this plane's fluxes: the ring of plane k + 1, the
      // raw fields of plane k + 2, the face fields of plane k + 1 and the old
      // values of what the update writes (converted and used before its
      // stores: a wait for loads would wait for stores issued after them)
      T rring[5], rrfb[3][2], rnext[5], rfb[3][2], uo[7];
#pragma unroll
      for (int c = 0; c < 5; ++c) rring[c] = T(1);
#pragma unroll
      for (int d = 0; d < 3; ++d) rrfb[d][0] = rrfb[d][1] = T(0);
      if (rwave) load_raw3<T>(U, bx(rx, ry, min(k + 1, kend)), bx.sy, bx.sz, rring, rrfb);
#pragma unroll
      for (int c = 0; c < 7; ++c) fz[c] = T(0);
      if (k >= z0) hlld7(zlo, ml[2], bn[2], gam, gm1_inv, fz);
#pragma unroll
      for (int c = 0; c < 7; ++c) zlo[c] = zhi[c];
      load_raw3<T>(U, bx(lx, ly, min(k + 2, kend + 1)), bx.sy, bx.sz, rnext, rfb);
#pragma unroll
      for (int s = 0; s < 7; ++s) uo[s] = ldb(U.f[s], ep);
      fb[0][0] = ldb(U.f[5], en);
      fb[0][1] = ldb(U.f[5], en, (int)sizeof(T));
      fb[1][0] = ldb(U.f[6], en);
      fb[1][1] = ldb(U.f[6], en + bx.sy);
      fb[2][0] = ldb(U.f[7], en);
      const unsigned mkn = fmask ? ldb(fmask, en / (unsigned)sizeof(T)) : 0u;
      if constexpr (kPark) {
        fx6p = sP[0][tid];
        fx6r = sP[0][tr];
        fy5p = sP[1][tid];
        fy5u = sP[1][tu];
        zl[1] = sF[14][tid];
        zl[2] = sF[15][tid];
      }
      __syncthreads();  // the face states have been read: the fluxes take their place
#pragma unroll
      for (int c = 0; c < 7; ++c) {
        sF[c][tid] = fx[c];
        sF[7 + c][tid] = fy[c];
      }
      if constexpr (kPark) {
        sP[0][tid] = fx[6];
        sP[1][tid] = fy[5];
      }
      sF[14][tid] = fz[5];
      sF[15][tid] = fz[6];
      if (rwave) {
        T wring[8];
        raw3_to_prim<T>(rring, rrfb, gm1, wring);
#pragma unroll
        for (int c = 0; c < 8; ++c) sW[c][rw] = wring[c];
      }
      __syncthreads();
      // edge EMFs: E_z at this lane's (cx - 1/2, cy - 1/2) corner of plane k
      // and at its high x and high y neighbours'; E_x at (cx, cy - 1/2) and
      // E_y at (cx - 1/2, cy) of z = k - 1/2 and those of the high y and high
      // x neighbours, from the inputs those lanes form theirs from
      const T fx5r = sF[5][tr], fx6n = sF[6][tr], fy6r = sF[13][tr];
      const T fx5u = sF[5][tu], fy5n = sF[12][tu], fy6u = sF[13][tu];
      const T ez0 = emf_mean(sF[5][td], fx[5], sF[13][tl], fy[6]);
      const T ezx = emf_mean(sF[5][tdr], fx5r, fy[6], fy6r);
      const T ezy = emf_mean(fx[5], fx5u, sF[13][tul], fy6u);
      const T ex = emf_mean(fy5p, fy[5], sF[15][td], fz[6]);
      const T ey = emf_mean(sF[14][tl], fz[5], fx6p, fx[6]);
      const T ey1 = emf_mean(fz[5], sF[14][tr], fx6r, fx6n);
      const T ex1 = emf_mean(fy5u, fy5n, fz[6], sF[15][tu]);
      fy5p = fy[5];
      fx6p = fx[6];
      fx6r = fx6n;
      fy5u = fy5n;
      if constexpr (kPark) zl[0] = sP[2][tid];
      T un[8];
      un[7] = bn[2] - curl_delta(cdx, ey1, ey, cdy, ex1, ex);
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        const int qx = hydro_comp(s, 0), qy = hydro_comp(s, 1), qz = hydro_comp(s, 2);
        un[s] = uo[s] - add_delta(up[s], cdz, fz[qz], zl[s]);
        // plane k's, up to the z-faces above it
        up[s] = flux_delta2<T>(cdx, sF[qx][tr], fx[qx], cdy, sF[7 + qy][tu], fy[qy]);
        zl[s] = fz[qz];
      }
      if constexpr (kPark) sP[2][tid] = zl[0];
      un[5] = uo[5] - minus_delta(up[5], cdz, ey, zl[5]);
      un[6] = uo[6] - delta_minus(cdz, ex, zl[6], up[6]);
      up[5] = face_delta2(cdy, ezy, ez0);
      up[6] = face_delta2(cdx, ezx, ez0);
      zl[5] = ey;
      zl[6] = ex;
      fb[2][1] = rfb[2][0];
      raw3_to_prim<T>(rnext, rfb, gm1, wnext);
      form_now(wnext);
      form_now(fb[0]);
      form_now(fb[1]);
      form_now(fb[2]);
      if (mk != 0u) {
        if ((mk & 1u) && own) st_flux7(F, 0, eb, fx);
        if ((mk & 2u) && own) st_flux7(F, 1, eb, fy);
        if ((mk & 4u) && k >= z0 && k < z1) st_flux7(F, 2, eb, fz);
      }
      mk = mkn & smask;
      // z-faces at k - 1/2 (element of plane k)
      if (ucell && k >= z0 && k < z1) stb(V.f[7], eb, un[7]);
      // cells and x-, y-faces of plane k - 1
      if (k - 1 >= z0 && k - 1 < z1 && k - 1 < uhz) {
        if (ucell)
#pragma unroll
          for (int s = 0; s < 5; ++s) stb(V.f[s], ep, un[s]);
        if (ubx) stb(V.f[5], ep, un[5]);
        if (uby) stb(V.f[6], ep, un[6]);
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
  // A persistent launch pays where its blocks come back for more.  With no more
  // claims than resident blocks each claim has a block of its own, as without the
  // queue: the blocks then reach the CUs one by one, while pops leave some CUs two
  // claims and some none (96^3 in FP64 in claims of two: 293 us from the queue,
  // 205 so; 258 while a CU held one block).
  const int claims = claim_blocks(nitems, claim, xcd);
  const bool per = q != nullptr && pblocks > 0 && claims > pblocks;
  const dim3 grid(per ? pblocks : claims);
  StatePair<T> SP;
  SP.s[0] = S0;
  SP.s[1] = S1;
#define AMR_FUSED_LAUNCH(K, THREADS) \
  hipLaunchKernelGGL((K), grid, dim3(THREADS), 0, s, grids, items, nitems, SP, parity, F, fmask, dt0, ph, err, q, xcd, claim)
  if (ndim == 3) {
    if (per) AMR_FUSED_LAUNCH((k_fused3<T, true>), 256);
    else AMR_FUSED_LAUNCH((k_fused3<T, false>), 256);
  } else {
    if (per) AMR_FUSED_LAUNCH((k_fused2<T, true>), 256);
    else AMR_FUSED_LAUNCH((k_fused2<T, false>), 256);
  }
#undef AMR_FUSED_LAUNCH
}

template <class T> int fused_occupancy(int ndim) {
  int a = 0;
  if (ndim == 3)
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, k_fused3<T, true>, 256, 0);
  else
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, k_fused2<T, true>, 256, 0);
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
