// Walk of a GEMM's output tiles by persistent workgroups, shared by the int8 and the binary16 tiled kernels.
#pragma once
#include "common.hpp"

namespace aweq {

struct TileWalk {
    int tiles_m, tiles_n, patch_m, patch_n, patches_n, n_patches;
    int n_ids;  // workgroup ids that may name a tile (whole rounds of patches over the XCDs)
    // the tile columns that do not fill a whole patch column form patches of their own shape
    int main_pn, n_main, tail_cols, tail_pm, per_patch, n_patches_fast;
    int strip_m, run;   // or (strip_m > 0) one sequence of tiles, `run` of it per XCD and round
};

// workgroup id -> output tile (false: the id names no tile).  Ids go round-robin over the XCDs,
// so id % 8 names the XCD; each XCD walks its own sequence of patch_m x patch_n patches.
// The last tile columns, when they do not fill a patch column, are walked as patches of their own
// shape (tail_pm x tail_cols, as many tiles as fit 32): a ragged patch would leave part of the XCD's
// workgroups without a tile, they would run ahead to their next id and the XCD's workgroups would
// stop walking K together, which is what lets them share operand panels in the L2.
__host__ __device__ __forceinline__ bool tile_of(const TileWalk& g, int vb, int& tile_m, int& tile_n)
{
    const int xcd = vb % kXcdCount, seq = vb / kXcdCount;
    if (g.strip_m) {
        const int l = ((seq / g.run) * kXcdCount + xcd) * g.run + seq % g.run;
        if (l >= g.tiles_m * g.tiles_n) return false;
        const int strip = l / (g.strip_m * g.tiles_n), in = l % (g.strip_m * g.tiles_n);
        const int height = min(g.strip_m, g.tiles_m - strip * g.strip_m);
        tile_m = strip * g.strip_m + in % height;
        tile_n = in / height;
        return true;
    }
    const int patch = (seq / g.per_patch) * kXcdCount + xcd;
    if (patch >= g.n_patches_fast) return false;
    const int within = seq % g.per_patch;
    if (patch < g.n_main) {
        const int pm = patch / g.main_pn, pn = patch % g.main_pn;
        tile_m = pm * g.patch_m + within % g.patch_m;
        tile_n = pn * g.patch_n + within / g.patch_m;
        return tile_m < g.tiles_m && tile_n < g.tiles_n;
    }
    if (within >= g.tail_pm * g.tail_cols) return false;
    tile_m = (patch - g.n_main) * g.tail_pm + within % g.tail_pm;
    tile_n = g.main_pn * g.patch_n + within / g.tail_pm;
    return tile_m < g.tiles_m;
}

// rounds of 256 workgroups the planned walk takes
inline int64_t rounds_of(const TileWalk& g) { return cdiv(g.n_ids, 256); }

// tile / patch plan of a launch on tiles of bm tokens x 256 channels; blocks: the grid of a kernel that takes one id per workgroup
inline int plan_walk(TileWalk& g, int64_t T, int64_t N, int64_t K, int bm, int64_t& blocks)
{
    const int64_t tiles_m = cdiv(T, bm), tiles_n = cdiv(N, 256);
    if (tiles_m * tiles_n > (1ll << 30)) return AWEQ_ERR_SHAPE;
    g.tiles_m = (int)tiles_m; g.tiles_n = (int)tiles_n;
    // patch of output tiles an XCD works on at a time: 32 tiles (one per compute unit), 8 (t) x 4 (n);
    // 4 x 8 when the contraction is long against N: the activation panels, the operand that does not
    // fit the memory-side cache, are then fetched half as often (1-2 % in the int8 GEMM; binary16, TFLOP/s: 1227 -> 1342 at
    // 4096 x 11008, 1236 -> 1342 at 4096 x 16384; 4096 x 4096 and 11008 x 4096 prefer 8 x 4)
    const int want_n = K >= 2 * N ? 8 : 4;
    g.patch_n = (int)(tiles_n < want_n ? tiles_n : want_n);
    g.patch_m = 32 / g.patch_n;
    if (g.patch_m > tiles_m) g.patch_m = (int)tiles_m;
    g.patches_n = (int)cdiv(tiles_n, g.patch_n);
    const int64_t patches_m = cdiv(tiles_m, g.patch_m);
    g.n_patches = (int)(patches_m * g.patches_n);
    const int64_t rounds = cdiv(g.n_patches, kXcdCount);
    blocks = rounds * kXcdCount * g.patch_m * g.patch_n;   // grid of the generic kernel
    if (blocks > 0x7fffffffll) return AWEQ_ERR_SHAPE;
    // the tiled kernel's walk: whole patch columns first, then the remaining tile columns as patches of their own
    g.per_patch = g.patch_m * g.patch_n;
    g.tail_cols = (int)(tiles_n % g.patch_n);
    g.main_pn = (int)(tiles_n / g.patch_n);
    g.tail_pm = g.tail_cols ? g.per_patch / g.tail_cols : 0;
    if (g.tail_cols && g.tail_pm > tiles_m) g.tail_pm = (int)tiles_m;
    g.n_main = (int)(patches_m * g.main_pn);
    g.n_patches_fast = g.n_main + (g.tail_cols ? (int)cdiv(tiles_m, g.tail_pm) : 0);
    g.n_ids = (int)(cdiv(g.n_patches_fast, kXcdCount) * kXcdCount * g.per_patch);   // <= blocks
    // One round of workgroups, or a few where patches leave so many ids without a tile that it costs another: the
    // tiles in one sequence, up and down strips of strip_m tile rows, an equal run of it for every XCD
    // (us, patches -> sequence: K = 4096: 1000 tokens x 4096 channels 34.8 -> 28.7, 2304 x 4096 59.7 -> 50.2, 2300 x 7168 88.8 -> 63.2)
    const int64_t tiles = tiles_m * tiles_n, ideal = cdiv(tiles, 256);
    g.strip_m = 0;
    if (ideal == 1 || (ideal <= 4 && rounds_of(g) > ideal)) {
        g.strip_m = want_n == 8 ? 4 : 8;
        g.run = ideal == 1 ? (int)cdiv(tiles, kXcdCount) : 32;
        g.n_ids = (int)(ideal * g.run * kXcdCount);
    }
    return AWEQ_OK;
}

// persistent launch: one workgroup per compute unit (a multiple of 8, so that id % 8 stays the XCD)
inline int launch_persistent(const void* fn, int threads, int lds, void* args, int64_t n_ids, hipStream_t st)
{
    int dev = 0, cus = 0;
    if (device_cus(dev, cus) != AWEQ_OK || raise_lds_limit(fn, dev, lds) != AWEQ_OK) return AWEQ_ERR_LAUNCH;
    void* argv[] = {args};
    int64_t grid = (cus / kXcdCount) * kXcdCount;
    if (grid < kXcdCount) grid = kXcdCount;
    if (grid > n_ids) grid = n_ids;
    if (hipLaunchKernel(fn, dim3((unsigned)grid), dim3((unsigned)threads), argv, lds, st) != hipSuccess) return AWEQ_ERR_LAUNCH;
    return launch_status();
}

}  // namespace aweq
