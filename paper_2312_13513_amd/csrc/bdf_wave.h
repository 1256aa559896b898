// Wave-per-cell and tile (16 lanes per cell) integrators (bdf_wave.hip):
// tables and launcher.
#pragma once

#include "chem_internal.h"
#include "wave_tables.h"

namespace chem {

// For each species k, the reactions with a non-zero net coefficient, in
// increasing reaction order: entries inc[inc_off[k] .. inc_off[k+1]) hold
// (reaction index, net coefficient).
struct WaveTables {
    const int *inc_off;
    const int2 *inc;
};

// Padded row count of the wave kernel for N unknowns (0 = unsupported).
int wave_kernel_rows(int N);

// The counts of a view, which the two decisions below read: species, reactions,
// pressure-dependent ones among them, bytes of the tables, and the reaction
// scratch per cell of the lane-group kernels.
void set_view_sizes(DevMechView &m, int K, int R, int n_pdep, int32_t table_bytes);

// Whether the wave (lanes = 64) or tile (lanes = 16) kernel of this mechanism
// keeps its reaction scratch (at most qstride doubles per cell in flight) in
// global memory because it does not fit in LDS.
bool wave_uses_global_scratch(const DevMechView &m, int lanes);

// Slices of that scratch (cells in flight) in `bytes` bytes, 64 to 4,096; 0 when
// no kernel the mechanism can run keeps its scratch in global memory.
int wave_scratch_slots(const DevMechView &m, size_t bytes);

// lanes = 64: one wave per cell (N <= 64); lanes = 16: four cells per wave
// (N <= 16).  qscratch holds max_groups slices of qstride doubles, used when the
// reaction scratch does not fit in LDS (wave_uses_global_scratch); the launch
// then runs at most max_groups groups, and fails if they fill no wave.
hipError_t launch_bdf_wave(const DevMechView &m, const WaveTables &wt, const Wave64Tables &w64, double *T, const double *p,
                           double *Y, int64_t ldY, int64_t n, double dt, const BdfParams &prm,
                           int32_t *status, int32_t *counters, unsigned long long *queue,
                           double *qscratch, int max_groups, bool fp32_lu, int lanes, hipStream_t s);

}  // namespace chem
