// cns_mixed.h -- launchers of the mixed form's kernels (cns_mixed.hip); all enqueue on
// bt.stream.
#pragma once

#include "cns_internal.h"

namespace cns {
namespace mixed {

int rows_for(int nx);                  // default rows per block of the x rows kernel
int rows_points(int nx, int rows);     // points per thread of the x rows kernel
void visc_fields(const Batch &bt, Launch L);
void viscous(const Batch &bt, Launch L);
void sweep_x(const Batch &bt, const Launch &L, bool visc);
void sweep_write(const Batch &bt, const Launch &L, int dir, bool visc);
void sweep_accum(const Batch &bt, const Launch &L, int dir, bool visc);
void sweep_rk(const Batch &bt, const Launch &L, bool visc);
// blocks per CU of the sweep with the update and of the viscous kernel (0: unknown)
int resident_sweep_blocks(int block);
int resident_tile_blocks();

}  // namespace mixed
}  // namespace cns
