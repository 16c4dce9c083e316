// Host functions that launch the kernels of the other translation units.
#pragma once
#include <hip/hip_runtime.h>

#include "pg_desc.h"

namespace pg {

// What every launch of an edge kernel takes.
struct EdgeLaunch {
    int threads, rank, lds;   // work-group size (one of kEdgeThreads), largest layer rank, LDS bytes
    unsigned tiles;
    hipStream_t stream;
    const EdgeTile *d_tiles;
    float *const *d_xs;
    int32_t *d_flags;
};
void launch_edge_round(const EdgeLaunch &l, const float *qin, float *qout, float *phat, int steps);
void launch_edge_pending(const EdgeLaunch &l, const ColDesc *cols, float *y, int64_t stride, bool from_y, const float *qin, float *qout,
                         const float *before, float *phat, int steps);
void launch_edge_iterate(const EdgeLaunch &l, float *q, float *pstate, float *uq, float *phat, int iterations, bool odd);
// y: where the matrices are read (null: in place); gs: gradients (null: none)
void launch_apply(int cols_compiled, unsigned ntiles, hipStream_t stream, const ApplyTile *tiles, const PairDesc *pairs, const ColDesc *cols,
                  float *const *xs, const float *y, int64_t stride, const float *right, const float *left, const float *const *gs, double eta);

void launch_apply_mixed(unsigned ntiles, hipStream_t stream, const MixedTile *tiles, const PairDesc *pairs, const ColDesc *cols,
                        float *const *xs, const float *y, int64_t stride, const float *right, const float *left, const float *const *gs, double eta);

// Edge sweeps.
struct SweepLaunch {
    int threads, rank, lds, nslots, reverse;
    hipStream_t stream;
    const SweepTile *tiles;
    const SweepDesc *descs;
    float *const *xs;
    float *qstate;
    double *part;
    float *phat;
    int32_t *flags;
};
void launch_sweep(const SweepLaunch &l);
void launch_sweep_finish(const SweepLaunch &l, const FinishTile *tiles, unsigned ntiles, bool long_rows);

}  // namespace pg
