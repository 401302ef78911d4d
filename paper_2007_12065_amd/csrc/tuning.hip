// Tile-shape table.  Defaults come from measurements on MI355X; the tuner
// replaces entries through pl_tune_set.
#include "tuning.h"
#include "tiles.h"

#include <algorithm>
#include <atomic>
#include <mutex>

namespace pl {

namespace {

std::mutex g_mu;
TileCfg g_cfg[kNumStages][kMaxRadius + 1] = {
    // Laplacian: {th, tw, fuse} per radius (3x3, 5x5: the fused path's
    // measured best on a 480x640 and a 128x2048 frame)
    {{0, 0, 0}, {16, 16, 4}, {16, 16, 2}, {8, 32, 1}, {8, 32, 1}},
    // bilateral (3x3: the region of the first sweep, 8 x 32, fills the threads;
    // 12 x 16 takes 35.0 us on a 480 x 640 frame, 6 x 30 33.7)
    {{0, 0, 0}, {6, 30, 2}, {2, 32, 1}, {8, 32, 1}, {8, 32, 1}},
    // batched Laplacian (a 64-frame mix)
    {{0, 0, 0}, {16, 16, 4}, {16, 16, 2}, {8, 32, 1}, {8, 32, 1}},
    // batched bilateral (3x3: 216 us for a batch of seven frames, 221 at 6 x 30)
    {{0, 0, 0}, {12, 16, 2}, {16, 16, 1}, {8, 32, 1}, {8, 32, 1}},
    // Laplacian, small frames (120x160, 64x1024)
    {{0, 0, 0}, {8, 16, 4}, {8, 16, 2}, {8, 32, 1}, {8, 32, 1}},
    // bilateral, small frames (3x3: cut to fewer rows where a frame has few
    // tiles, bil_frame_tile)
    {{0, 0, 0}, {6, 30, 2}, {2, 32, 1}, {4, 16, 1}, {4, 16, 1}},
};

// gfx950 LDS per workgroup, less room for the batched kernels' static LDS
constexpr size_t kLdsMax = 156 * 1024;

}  // namespace

size_t cfg_lds_bytes(Stage s, int R, TileCfg c) {
    return is_laplacian(s) ? lap_lds_bytes(R, c.fuse, c.th, c.tw)
                           : bil_lds_bytes(R, c.fuse, c.th, c.tw, bil_waves(R, s == kStageBatchBilateral));
}

TileCfg bil_launch_tile(int R, TileCfg c, int F) {
    if (!bil_in_place(R, c.fuse, c.th, c.tw) || F >= c.fuse) return c;
    const int grow = 2 * R * (c.fuse - std::max(F, 1));
    return TileCfg{c.th + grow, c.tw + grow, c.fuse};
}

TileCfg bil_frame_tile(int R, TileCfg c, int F, int Mq, int Nq) {
    if (!bil_in_place(R, c.fuse, c.th, c.tw)) return c;
    auto per_cu = [&](const TileCfg &cfg) {
        const TileCfg t = bil_launch_tile(R, cfg, F);
        const long tiles = (long)((Mq + t.th - 1) / t.th) * ((Nq + t.tw - 1) / t.tw);
        return (tiles + kNumCu - 1) / kNumCu;
    };
    TileCfg best = c;
    for (const TileCfg &t : {TileCfg{c.th * 2 / 3, c.tw + 2, c.fuse}, TileCfg{c.th / 2, c.tw + 2, c.fuse}})
        if (t.th > 0 && t.th < best.th && bil_in_place(R, t.fuse, t.th, t.tw) && per_cu(t) <= per_cu(best))
            best = t;
    return bil_launch_tile(R, best, F);
}

TileCfg tile_cfg(Stage s, int R) {
    std::lock_guard<std::mutex> g(g_mu);
    return g_cfg[s][R];
}

bool set_tile_cfg(Stage s, int R, TileCfg c) {
    if (R < 1 || R > kMaxRadius || c.th < 1 || c.tw < 1 || c.fuse < 1 || c.fuse > 8) return false;
    if (c.th * c.tw > 64 * kTileBlock) return false;
    if (cfg_lds_bytes(s, R, c) > kLdsMax) return false;
    std::lock_guard<std::mutex> g(g_mu);
    g_cfg[s][R] = c;
    return true;
}

pl_status allow_lds(const void *kernel, size_t bytes) {
    if (bytes <= 64 * 1024) return PL_OK;
    return hip_check(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)bytes),
                     "hipFuncSetAttribute");
}

}  // namespace pl
