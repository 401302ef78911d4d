// Runtime tile shapes and sweep fusion, read by every launcher and set by the
// tuner (pl_tune_set).  The only mutable global state of the library.
#pragma once

#include "common.h"

namespace pl {

enum Stage {
    kStageLaplacian = 0,
    kStageBilateral = 1,
    kStageBatchLaplacian = 2,      // the batched path's entries
    kStageBatchBilateral = 3,
    kStageLaplacianSmall = 4,      // single frames of at most kSmallFramePoints points
    kStageBilateralSmall = 5,
    kNumStages = 6
};
inline bool is_laplacian(Stage s) {
    return s == kStageLaplacian || s == kStageBatchLaplacian || s == kStageLaplacianSmall;
}
// Single frames up to this many points read the *Small entries: a 64 x 1024
// frame has a quarter of the tiles of a 480 x 640 one, and the shapes that
// fill the chip differ.
constexpr long kSmallFramePoints = 1L << 17;
inline Stage frame_stage(bool laplacian, int M, int N) {
    const bool small = (long)M * N <= kSmallFramePoints;
    if (laplacian) return small ? kStageLaplacianSmall : kStageLaplacian;
    return small ? kStageBilateralSmall : kStageBilateral;
}
constexpr int kMaxRadius = 4;                 // kernel sizes 3, 5, 7, 9

struct TileCfg {
    int th, tw;      // tile rows x columns (points for the Laplacian, quads for the bilateral)
    int fuse;        // sweeps fused per launch
};

// Tile of a bilateral launch of F of the c.fuse sweeps (the last launch may have
// fewer): where they run in place, it grows by the halo it does not need, so
// that every thread keeps a quad.
TileCfg bil_launch_tile(int R, TileCfg c, int F);
// The same for a single frame of Mq x Nq quads.  Tiles of an in-place shape may
// first be cut to two thirds or half of their rows (6 x 30 quads to 4 x 32 or
// 3 x 32): of the three the one that gives a CU the fewest tiles, then the one
// of fewest rows (a small frame's launch takes as long as the CU with the most
// rows).  Frames of four and two sweeps, us (tiles of the fullest CU) at 6, 4
// and 3 rows: 120 x 160 15.1 (1), 14.2 (1), 13.6 (1); 200 x 220 17.2 (2), 16.6
// (2), 16.1 (2); 200 x 300 18.5 (2), 17.1 (2), 17.4 (3); 240 x 320 18.1 (2),
// 19.5 (3), 19.3 (4); 64 x 1024 17.6 (2), 17.0 (2), 17.2 (3).  Two rows or 5 x
// 30 are best at few sizes and by little (120 x 160 14.1 and 14.3).
TileCfg bil_frame_tile(int R, TileCfg c, int F, int Mq, int Nq);

// Current configuration for a stage and window radius (1..4).
TileCfg tile_cfg(Stage s, int R);
// Replace it; returns false if the shape does not fit the kernels' limits.
bool set_tile_cfg(Stage s, int R, TileCfg c);
// LDS bytes a configuration needs.
size_t cfg_lds_bytes(Stage s, int R, TileCfg c);
// Raise a kernel's dynamic-LDS limit when a configuration needs more than
// the default 64 KB (once per kernel and size).
pl_status allow_lds(const void *kernel, size_t bytes);

}  // namespace pl
