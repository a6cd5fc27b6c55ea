// Fused FP64 envelope stages: when a plan takes them, their tiles and their launch.
#pragma once

#include "fdetd_internal.h"

#if defined(__HIPCC__)
#define FDETD_ENV_HD __host__ __device__
#else
#define FDETD_ENV_HD
#endif

namespace fdetd {

// Blocks of kEnvWaves wavefronts side by side along z run env_depth consecutive stages in one pass.  Depth 4 only
// at N_D = 1: the windows and delay lines of the stages stand in registers, and 4 stages at N_D = 2 already take
// the 256 of two wavefronts per SIMD (order 4, 4096 x 512: 89 us per 4 stages with depth 2, 106 with depth 4).
// From N_D = 5 on the march stage by stage is the faster one (order 12, 4096 x 512: 152 us per 4 stages, 171 fused;
// order 16: 161, 257): the rows that a block forms for its neighbours grow with N_D while the bytes saved do not.
// FP64 only, where the groups give the same bits as the single stages: the FP32C rows next to the axis, in FP64
// arithmetic, would reach (S - 1) N_D rows further.
constexpr int kEnvWaves = 4;
constexpr int kEnvBlocks = 512;           // blocks that run at a time: two per CU
constexpr int kEnvFuseND = 4;
// Fewest cells of a launch that takes groups, or (autotuned plans) times them against the single stages.  us per
// step of 4 stages one by one | fused, in calls of 1 and of 2 steps:
//                  order 2         order 4         order 6         order 8
//   1400 x 180   30 | 35 27      32 | 32 32      32 | 37 38      34 | 38 41
//   2048 x 256   44 | 44 29      45 | 43 41      46 | 45 43      48 | 50 52
//   2400 x 300   56 | 49 34      58 | 50 42      59 | 55 49      60 | 57 54
//   2900 x 360   72 | 61 40      75 | 66 55      77 | 69 60      79 | 76 70
// (the waves of a small launch wait for the longest march, whatever it saves)
constexpr size_t env_fuse_cells(int nd) { return nd <= 3 ? 1 << 19 : 700000; }
constexpr int kEnvColumns = (1 << 27) - 1;  // widest grid: the bytes of a row are an int
constexpr int kEnvRows = 640;  // most rows of a march (output rows, and the rows before and behind them)
constexpr int env_depth(int nd) { return nd == 1 ? 4 : 2; }
constexpr int env_out_columns(int nd) { return kEnvWaves * 32 - 2 * (env_depth(nd) - 1) * nd; }
// Arguments of a group's launch: those of a stage (psi, aux, chi: the caller's planes) and more.  The FP64 stage
// launches of fdetd_march.hip hand them on to launch_envelope_fused by their role.
constexpr int ROLE_ENV_GROUP = 3;
struct EnvFuseArgs : BatchArgs {
    int seg;                       // rows per segment
    int sel_in, sel_psi, sel_out;  // vectors of the group: 0 the caller's planes, 1, 2 the plan's stage vectors
    double coefs[4];               // of the group's stages, in order
    int begin[kMaxBatch];          // first tile of each problem
};
hipError_t launch_envelope_group(int nd, EnvFuseArgs a, hipStream_t s);  // dispatch on nd (fdetd_dispatch.cpp)
hipError_t launch_envelope_fused(int nd, const EnvFuseArgs &a, hipStream_t s);

// A tile: first output column, output rows.  Tile r of an nz x nr grid: oc output columns per tile, seg rows per
// segment, strips numbered fastest.
struct FuseTile {
    int o0, k0, k1;
};
FDETD_ENV_HD inline int fused_tiles(int nz, int nr, int seg, int oc) { return (nz + oc - 1) / oc * ((nr + seg - 1) / seg); }
FDETD_ENV_HD inline bool decode_fused(int nz, int nr, int r, int seg, int oc, FuseTile &c)
{
    const int ns = (nz + oc - 1) / oc, sl = r / ns;
    c.o0 = (r - sl * ns) * oc;
    c.k0 = sl * seg;
    c.k1 = c.k0 + seg < nr ? c.k0 + seg : nr;
    return r >= 0 && c.o0 < nz && c.k0 < c.k1;
}

// Rows per segment for the `count` grids of a batch, and the tiles they give: a block marches the segment and the
// rows before its first one, kEnvBlocks blocks at a time.  False where a group cannot take one of the grids.
inline bool env_tiling(int nd, int count, const int *nz, const int *nr, int &seg, int &tiles)
{
    const int lag = (env_depth(nd) - 1) * nd, oc = env_out_columns(nd);
    for (int t = 0; t < count; ++t)
        if (nz[t] > kEnvColumns) return false;
    long long least = -1;
    for (int s = 8; s + 3 * lag + 4 <= kEnvRows; ++s) {
        long long blocks = 0;
        for (int t = 0; t < count; ++t) blocks += fused_tiles(nz[t], nr[t], s, oc);
        const long long cost = (blocks + kEnvBlocks - 1) / kEnvBlocks * (s + 2 * lag + 4);
        if (least < 0 || cost < least) {
            least = cost;
            seg = s;
            tiles = (int)blocks;
        }
    }
    return true;
}

}  // namespace fdetd
