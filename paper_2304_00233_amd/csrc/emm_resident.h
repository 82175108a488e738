// Whole time loops in one launch, for grids whose state fits on the chip.
#pragma once

#include "emm_internal.h"
#include "emm_resident_plan.h"

#include <vector>

namespace emm {

// A stretch of one grid row that receiver stencils read: x0 <= i < x0 + len
// of component comp at (y, z), kept at offset off of a step's samples.
struct ResidentRow {
    int comp, y, z, x0, len, off;
};

// What a model grants its resident runs; tests tighten it (emm_test_resident)
// to send a run the way back to half-step launches.
struct ResidentLimits {
    unsigned long long patience = 200000000ull;   // a wait: ticks of the 100 MHz wall clock
    int launches = -1;                            // cooperative launches (-1: any number)
};

struct ResidentParams {
    int gy, gz, ty, tz, groups;       // as in the plan
    unsigned long long *mail;         // [6][n3][n2][pitch] words (tag << 32 | value) of tile edges
    unsigned tag;                     // tag of this launch's first half step; each counts one up
    int n0, n1;                       // time steps [n0, n1)
    int src;                          // source
    // receiver samples [n - nbase][per_step]: rows of H (read in the E step)
    // and E (in the H step)
    const ResidentRow *rows[2];
    int nrows[2];
    float *samples;
    int nbase, per_step;
    // items of one source (item q of the source is item q * nsrc + src of
    // its list): offset of the samples of stencil row (c, b), [item][(2r)^2],
    // -1 for a row off the update set (zeros)
    const int *item_rows[2];
    int nitems[2];
    float *snap;                      // not null: E after step n also goes to snap + (n - n0) * snap_stride
    long long snap_stride;
    int *stuck;                       // set when a wait ran out of time (the run is then void)
    unsigned long long patience;      // wall-clock ticks a wait may take
};

// One cooperative launch of steps [n0, n1) for one source: state from pe / ph
// field and CPML arrays and back to them.
hipError_t launch_resident(int r, const ResidentPlan &plan, const StepParams &pe, const StepParams &ph,
                           const ResidentParams &x, hipStream_t s);

// DTFT of the samples of steps [n0, n1): u (double [n - nbase][items]) is
// scratch.
void launch_resident_dft(int r, const StepParams &pe, const StepParams &ph, const ResidentParams &x, double *u,
                         hipStream_t s);

}  // namespace emm
