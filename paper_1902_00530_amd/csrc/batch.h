// Device-side tables of a batched sweep, shared by its kernels' source files.
#pragma once

#include "internal.h"

namespace lbm {

struct BatchTile {
    int32_t lat;
    int16_t tx, ty;
};

struct LatDesc {
    StepArgs a;
    void *buf[2];
    float B;            // CIL B for zeta
    int32_t mt_begin;   // first moments tile
    int32_t mt_count;   // moments tiles of this lattice
    int32_t nrb;        // moments row blocks
    int64_t col_off;    // offset of this lattice's column partials
    int64_t cm_off;     // offset of this lattice's column means
    float add;          // added to every population after each sample (drho / Q)
    int32_t stream;     // 1: stores streamed past the caches (two buffers beyond the
                        // Infinity Cache budget: the lattice is a group of its own)
};

struct MomTile {
    int32_t lat;
    int16_t cx, cy;
};

struct Ctrl {
    int64_t t0;      // absolute step index of the next step
    int64_t k0;      // steps done in this sweep (buffer parity)
    int64_t sample;  // index of the next sample
    int64_t pad;
};

// Several steps per launch over a list of g.tx x g.ty tiles (multi.h; D2Q9: F32
// storage only); step_off: steps of this chunk before the launch, launch_off:
// launches before it (the buffer parity).
hipError_t launch_batch_multi(int lattice, int model, int storage, int flags, const MultiGeom &g, int64_t ntiles,
                              const BatchTile *tiles, const LatDesc *lats, const Ctrl *ctrl, int step_off,
                              int launch_off, hipStream_t s);

}  // namespace lbm
