// asd_pair.h -- the two faces of a multiscale window in one launch (the
// coupled multiscale step moves data across both x faces every step; the
// launches, not the bytes, dominate there).  Library-internal: not part of
// the C ABI.
#pragma once

#include "asd.h"
#include "asd_internal.h"

namespace asd {

// what a micromagnetic region shows and takes at the x face beside the window
struct RegionFace {
    double *ghost;            // its face neighbours [ny nz][3], written
    const void *m;            // its magnetisation [3][n], FP64 (elem 8) or FP32
    int64_t n;
    int32_t elem, nx, col;    // cells per row, the face's cell in a row
#ifdef __HIPCC__
    __device__ double at(int64_t cell, int d) const
    {
        return elem == 8 ? ((const double *)m)[d * n + cell] : (double)((const float *)m)[d * n + cell];
    }
#endif
};

// both sides of a window: its boundary strips (one coarse column each), the
// frozen columns beside it and the regions
struct WindowFaces {
    TransferArgs strip[2], cols[2];
    RegionFace region[2];
    int32_t gx, layers, col_blocks;  // filled by launch_window_faces
};
int launch_window_faces(WindowFaces &f, void *stream);

// the exchange of directions across both faces of the window [org, org + nx) of
// system s with coarse cells cx x cy x cz: asd_coarse_grain of its first and
// last coarse column into the regions' face neighbours (as asd_mm_set_face), the
// regions' face cells (as asd_mm_get_face) into the cx columns beside the window
// (as asd_set_columns), in one launch; same checks and error codes
int window_faces(asd_t *h, int32_t s, int32_t org, int32_t nx, int32_t cx, int32_t cy, int32_t cz,
                 const RegionFace &left, const RegionFace &right);
// the handle's time step and lattice cell edges (x, y: a; z: a for SC, c for
// L1_0), for the checks of the multiscale window
void lattice_cell(const asd_t *h, double *dt, double edge[3]);
// the atomic moment mu_s (J/T) of the handle
double atom_moment(const asd_t *h);
// stored columns of track system s (0 for a system without a track or a bad index)
int32_t track_columns(const asd_t *h, int32_t s);
// the demagnetising mesh of a handle: coarse cell (lattice cells) and cells
// per axis; ASD_ESTATE when the handle has no demagnetising field
int demag_mesh(const asd_t *h, int32_t cell[3], int32_t mesh[3]);
// the field (T) that system s adds per coarse cell at both Heun stages in
// place of the frozen track's stray field: cells [off, off + ncx) of a wider
// mesh of src_nx cells along x (src [3][src_nx ncy ncz], device, FP64),
// copied now; clear_cell_field goes back to the track's stray field
int set_cell_field(asd_t *h, int32_t s, const double *src, int32_t src_nx, int32_t src_off);
int clear_cell_field(asd_t *h);
}  // namespace asd
