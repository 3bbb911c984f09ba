// grid_device.h -- the refined grid and its brick layout built on the GPU
// (Secs. 4.3-4.4 construction, Sec. 8 remeshing without the host tree
// build).  The result is the same HostGrid and DeviceLayout, value for
// value, as build_grid + build_layout produce on the host.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <string>

#include "grid_builder.h"
#include "layout.h"
#include "lattice.h"

namespace lbm {

// device memory for the builder's temporaries (released before return)
struct DevAlloc {
  void *(*alloc)(size_t bytes, void *ctx);
  void (*release)(void *p, void *ctx);
  void *ctx;
};

// The grid as the caller keeps it on the device (allocated through the
// DevAlloc, owned by the caller): the canonical tables and the lists over
// slots that the update reads.  The per-cell tables of the HostGrid and the
// DeviceLayout then stay empty; fetch_host_grid and fetch_host_layout copy
// them when a host reader asks (grid exports, inflow noise, in-place
// builds).  Copying them on every build and the slot lists back up was most
// of a remesh: 1024^2 vortex with four steps, 11.2 -> 3.9 ms.
// The caller may release nbr once it has formed the per-slot flags.
struct DeviceGridArrays {
  // canonical
  int32_t *xyz = nullptr;     // [n][3]
  int8_t *lev = nullptr;      // [n]
  uint8_t *flag = nullptr;    // [n] canonical flags
  int32_t *nbr = nullptr;     // [Q-1][n] canonical values
  int32_t *slot_of = nullptr; // [n]
  int32_t *ghost = nullptr, *child = nullptr;      // [ng], [ng][2^D]
  uint64_t *unknown = nullptr;                     // [ng]
  int32_t *bc_cell = nullptr, *bc_src = nullptr;   // [nbc]
  int8_t *bc_face = nullptr;                       // [nbc]
  int64_t n = 0, ng = 0, nbc = 0;
  int Qm = 0, nch = 0;
  // brick layout (DeviceLayout's tables)
  int32_t *cell_of = nullptr, *nbrick = nullptr, *xbase = nullptr, *xnbr = nullptr;
  unsigned long long *xmask = nullptr;
  uint64_t *xreg = nullptr;                        // regular_pulls
  int64_t nslot = 0, xstride = 0;
  int nbp = 0;
  // lists over slots and explicit rows
  int32_t *ghost_slot = nullptr, *child_slot = nullptr, *child_row = nullptr;
  int32_t *row_ghost = nullptr;                    // [rows] ghost of a row, or -1
  int32_t *bc_cell_slot = nullptr, *bc_src_slot = nullptr;
  double *sigma = nullptr, *rho_inf = nullptr;     // [nslot], null without a sponge
  int64_t rows[8] = {0}, sponge[8] = {0};          // explicit rows and sponge cells per level
};

// Same arguments and validation as build_grid (periodic[a]: both faces of
// axis a are periodic).  Returns 0, -1 (argument error), -2 (mask error) or
// -3 (device allocation or runtime failure); *err receives the text.
// keep (may be null) receives the device tables above; without it every
// table comes back in g and y.  Synchronises the stream.
int build_grid_device(const LatticeInfo &lat, int dim, const int32_t ext[3], int L, const MaskView *refine,
                      const MaskView *solid, const FaceSpec faces[6], const bool periodic[3], const DevAlloc &da,
                      hipStream_t stream, HostGrid *g, DeviceLayout *y, DeviceGridArrays *keep, std::string *err);

// The host copies of a kept grid's tables that are not there yet: everything
// of *g but nbr and the sponge fields, everything of *y.
int fetch_host_grid(const DeviceGridArrays &dg, HostGrid *g, hipStream_t stream, std::string *err);
int fetch_host_layout(const DeviceGridArrays &dg, DeviceLayout *y, hipStream_t stream, std::string *err);

// per-slot device flags: the canonical flag, F_MOVING where a population is
// pulled from a moving wall, F_HOLE for slots without a cell
void launch_slot_flags(const DeviceGridArrays &dg, int64_t nslot, uint8_t *out, hipStream_t stream);

// flags[slot[k]] |= bit for m distinct slots
void launch_mark_slots(const int32_t *slot, int64_t m, uint8_t bit, uint8_t *flags, hipStream_t stream);

// remesh_sources on the device: for every cell of `nw` its sources among
// the flow cells (not fine ghosts) of `old`, same order and weights value
// for value, from the two grids' kept device tables (coordinates, levels,
// flags).  *off [n_new + 1], *src, *wt are device arrays from `da` that
// the caller releases.  Returns 0, -1 with *err set when a new cell covers
// no old flow cell (the lowest such cell is named), -3 on a device failure.
int remesh_sources_device(const HostGrid &old, const DeviceGridArrays &dold, const HostGrid &nw,
                          const DeviceGridArrays &dnew, const DevAlloc &da, hipStream_t stream, int64_t **off,
                          int32_t **src, double **wt, std::string *err);

}  // namespace lbm
