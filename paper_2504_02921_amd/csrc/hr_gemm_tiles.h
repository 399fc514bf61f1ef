// The order in which the workgroups of a projection take its tiles: shared by the GEMM kernels and by the kernel that brings their
// weights into the L2s ahead of them.  Device code.
#pragma once

#include <hip/hip_runtime.h>

#include "hr_kernels.h"

namespace hr {

constexpr int kXcds = 8, kGroupM = 8;

struct TileCoord { int tm, tn, share, shares; bool valid; };     // tile; its number among the `shares` that follow each other in one tile column

// Workgroup ids are dealt round-robin over the XCDs: XCD x works on tiles x * per_xcd .. (x + 1) * per_xcd - 1
__device__ __forceinline__ TileCoord tile_at(int tile, int tiles_m, int tiles_n) {
    TileCoord c;
    const int width = kGroupM * tiles_n;
    const int group = tile / width;
    const int first_m = group * kGroupM;
    const int gsz = min(tiles_m - first_m, kGroupM);
    const int in = tile - group * width;
    c.valid = true;
    c.share = in % gsz;
    c.shares = gsz;
    c.tm = first_m + c.share;
    c.tn = in / gsz;
    return c;
}

__device__ __forceinline__ TileCoord map_tile(int pid, int tiles_m, int tiles_n) {
    const int n_tiles = tiles_m * tiles_n;
    const int per_xcd = (n_tiles + kXcds - 1) / kXcds;
    const int tile = (pid % kXcds) * per_xcd + pid / kXcds;
    TileCoord c = tile_at(tile, tiles_m, tiles_n);
    c.valid = tile < n_tiles && pid / kXcds < per_xcd;
    return c;
}

// The workgroups behind the `first`-th of a launch with idle CUs do not take part in it: they touch the weights that the next
// launches read, XCD by XCD in the order above, 64 bytes per lane, so that those find them in their XCD's L2 (what a kernel read
// stays there for the next: 256 workgroups reading 8 MB take 1.5 us from HBM, 0.65 from their own L2 and 1.5 from
// another XCD's reading).  NW: wavefronts of a workgroup; lds: room for 256 bytes for each of them, read by nobody.
template <int NW>
__device__ __forceinline__ void warm_weights(const WeightWalks& ws, int first, char* lds) {
    typedef __attribute__((address_space(3))) void* lds_p;
    typedef const __attribute__((address_space(1))) void* gbl_p;
    const int xcd = (int)blockIdx.x % kXcds;
    const int skip = ((xcd - first) % kXcds + kXcds) % kXcds;            // first + skip: the first such workgroup on this XCD
    const int me = ((int)blockIdx.x - first - skip) / kXcds, all = ((int)gridDim.x - first - skip + kXcds - 1) / kXcds;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int i = 0; i < ws.n; ++i) {
        const WeightWalk& w = ws.w[i];
        const int n_tiles = w.tiles_m * w.tiles_n, per = (n_tiles + kXcds - 1) / kXcds;
        int last = -1;
        for (int t = xcd * per; t < min((xcd + 1) * per, n_tiles); ++t) {
            const TileCoord c = tile_at(t, w.tiles_m, w.tiles_n);
            if (c.tn == last) continue;                                  // the tiles of a column follow each other
            last = c.tn;
            const char* base = w.W + (size_t)c.tn * w.bn * w.row_bytes;
            const int bytes = min(w.bn, w.rows - c.tn * w.bn) * w.row_bytes;      // whole rows: one run of memory
            for (int off = (me * NW + wave) * 4096 + lane * 64; off < bytes; off += all * NW * 4096)
                __builtin_amdgcn_global_load_lds((gbl_p)(base + off), (lds_p)(lds + wave * 256), 4, 0, 0);
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);              // nothing is on its way into LDS when the wave ends
}

}  // namespace hr
