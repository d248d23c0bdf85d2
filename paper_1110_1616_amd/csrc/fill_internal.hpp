// Internal fill / CFL / marshalling types and launchers of libamrmhd.so.
#pragma once
#include "amr_internal.hpp"

namespace amr {

// Band element copy: pool element dst takes the value of element src.  The
// map of one fill lists cells first, then x-, y- and z-faces; int4 class
// bounds give the end of each group.
struct CopyEntry {
  int32_t dst;
  int32_t src;
};

// Band element prolongation from the parent level (see the kernels for the
// meaning of `code`, below bit kProlongRow).  src is the coarse element.  The
// parent grid's strides come with the entry, not with a load of the grid that
// the loads of its fields would wait for: in 3-D the row length P[0] in the
// code's bits from kProlongRow (element indices have 31 bits and the other two
// extents are at least 6, so it has less than 26) and the plane size
// P[0] P[1] in `stride`; in 2-D the row length in `stride`.
struct ProlongEntry {
  int32_t dst;
  int32_t src;
  int32_t stride;
  int32_t code;
};
constexpr int kProlongRow = 5;
inline ProlongEntry prolong_entry(int64_t dst, int64_t src, const GridDesc& P, int nd, int code) {
  if (nd == 2) return ProlongEntry{(int32_t)dst, (int32_t)src, P.P[0], code};
  return ProlongEntry{(int32_t)dst, (int32_t)src, P.P[0] * P.P[1], code | (P.P[0] << kProlongRow)};
}
template <int NDIM> __host__ __device__ inline void prolong_strides(const ProlongEntry& e, int64_t (&st)[3]) {
  st[0] = 1;
  st[1] = NDIM == 3 ? e.code >> kProlongRow : e.stride;
  st[2] = NDIM == 3 ? e.stride : 0;
}
// Cell widths of a level, evaluated as the device kernels do.
template <class T> struct Widths {
  T w[3];
};
template <class T> Widths<T> level_widths(const Phys& ph, int ndim, int level) {
  double rl = 1.0;
  for (int l = 0; l < level; ++l) rl *= (double)ph.ratio;
  return Widths<T>{{T(ph.dx0[0] / rl), T(ph.dx0[1] / rl), T(ndim == 3 ? ph.dx0[2] / rl : 1.0)}};
}

template <class T>
void launch_copy(int ndim, const CopyEntry* ent, int n, int4 cls, DevState<T> U, hipStream_t s);
// A full band fill (the copies and both prolongations) in one launch.
template <class T>
void launch_fill_full(int ndim, const CopyEntry* cp, int nc, int4 cls, const ProlongEntry* cells, int ncells,
                      const ProlongEntry* faces, int nfaces, DevState<T> Us, DevState<T> Ud, Phys ph, int plevel,
                      hipStream_t s);
// Prolongation reads the parent level (plevel) from Us and writes the band
// into Ud.
template <class T>
void launch_prolong(int ndim, const ProlongEntry* cells, int ncells, const ProlongEntry* faces, int nfaces,
                    DevState<T> Us, DevState<T> Ud, Phys ph, int plevel, hipStream_t s);
template <class T>
void launch_cfl(int ndim, const GridDesc* grids, const int4* items, int nitems, DevState<T> S0, DevState<T> S1,
                uint32_t parity, Phys ph, unsigned long long* acc, ErrBlock* err, double cfl, double* dt0,
                hipStream_t s);
template <class T>
void launch_load_prim(int ndim, const GridDesc& G, const double* const* prim, const double* const* b,
                      DevState<T> U, double gamma, hipStream_t s);
template <class T>
void launch_store(int ndim, const GridDesc& G, DevState<T> U, double* const* out, hipStream_t s);

}  // namespace amr
