// SAP domain solves kept on the chip: one launch per colour and cycle forms
// the SAP residual of every domain, runs its nmr minimal-residual steps and
// adds the result to psi (Sec. 2.2).  A domain and a group of columns (a
// unit) belong to one workgroup, or to G workgroups that own a tile of the
// domain each and exchange tile faces and partial sums through memory.
#pragma once

#include "internal.h"

namespace mbbs {

// Storage of eta and psi on this path, complex element of (position D of the
// domain in domain-major order, column group cg, tile, component e, site of
// the tile, column c of the group):
//   ((((D ncg + cg) G + tile) 12 + e) ts + site) lg + c
// so that a workgroup reads and writes whole runs.
struct DomPlan {
  int t[4];         // tile extents (each divides the SAP block extent)
  int nt[4];        // tiles per domain and direction
  int tstr[4];      // strides of the site index inside a tile
  int tgs[4];       // strides of the tile index inside a domain
  int n[4];         // entries (site, column chunk) of a tile face
  int hoff[4][2];   // first halo entry of direction m from the tile below [0] / above [1]
  int ts;           // sites per tile
  int lg;           // columns per unit (divides L)
  int C;            // columns per thread
  int np;           // column chunks per site: lg / C
  int T;            // threads per workgroup: ts np
  int TS;           // cells per LDS row (256 or 512), at least T
  int G;            // workgroups (tiles) per unit
  int ncg;          // column groups: L / lg
  int H;            // halo entries of a tile
  int units;        // domains of one colour x ncg
  int ngroups;      // workgroup groups of a launch (G > 1)
};

// Whether (and how) SAP with MR domain solves of nmr steps runs on this path for
// the lattice, L, precision and workspace.
bool dom_plan(const mbbs_lattice_s* lat, const SapBuffers& b, int nmr, DomPlan* out);
// The same for any 16-byte aligned workspace with `room` bytes in r and w.
bool dom_plan(const mbbs_lattice_s* lat, int L, int prec, int nmr, size_t room, DomPlan* out);
// psi = M eta on the path of `p`: in (FP64 lexicographic, times gam if given)
// to out.  The workspace is bound as for the other SAP kernels.
int dom_sap_apply(const mbbs_lattice_s* lat, const SapBuffers& b, const DomPlan& p, int ncy, int nmr,
                  const double2* in, const double2* gam, double2* out, const int* frozen, hipStream_t st,
                  struct Profiler* prof);

// FP64 lexicographic block (times gam if given) <-> the storage of `p` in FP64
// or FP32.  order: the local sites in storage order (null: as the tiles of `p`
// have them).  dom_to also clears nclear words; dom_from writes NaN to all of
// `out` if the word *lost (null: none) is set.
int dom_to(const mbbs_lattice_s* lat, int prec, int L, const DomPlan& p, const int* order, const double2* in,
           const double2* gam, void* out, unsigned* clear, int nclear, const int* frozen, hipStream_t st);
int dom_from(const mbbs_lattice_s* lat, int prec, int L, const DomPlan& p, const int* order, const void* in,
             double2* out, const int* lost, const int* frozen, hipStream_t st);

}  // namespace mbbs
