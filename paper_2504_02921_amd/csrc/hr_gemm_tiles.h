// The order in which the workgroups of a projection take its tiles: shared by the GEMM kernels and by the kernel that brings their
// weights into the L2s ahead of them.
#pragma once

#include "hr_layout.h"

namespace hr {

constexpr int kXcds = 8, kGroupM = 8;
// how many tiles of a column take turns reading W ahead at least
constexpr int kAheadShares = 4;

struct TileCoord { int tm, tn, share, shares; bool valid; };     // tile; its number among the `shares` that follow each other in one tile column

// Tiles come in groups of kGroupM rows of tiles (the last group has what is left), column after column.  Workgroup ids are dealt
// round-robin over the XCDs: XCD x works on tiles x * per_xcd .. (x + 1) * per_xcd - 1
HR_HD TileCoord map_tile(int pid, int tiles_m, int tiles_n) {
    const int n_tiles = tiles_m * tiles_n;
    const int per_xcd = (n_tiles + kXcds - 1) / kXcds;
    const int tile = (pid % kXcds) * per_xcd + pid / kXcds;
    TileCoord c;
    c.valid = tile < n_tiles && pid / kXcds < per_xcd;
    const int width = kGroupM * tiles_n;
    const int group = tile / width;
    const int first_m = group * kGroupM;
    const int gsz = tiles_m - first_m < kGroupM ? tiles_m - first_m : kGroupM;
    const int in = tile - group * width;
    c.share = in % gsz;
    c.shares = gsz;
    c.tm = first_m + c.share;
    c.tn = in / gsz;
    return c;
}

// The tile columns [c0, c1) that tiles [t0, end) of one group touch, t0 .. t1 - 1 being an XCD's tiles that are left.  near: they are worth
// reading ahead: a last group of fewer than kAheadShares rows of tiles lies on one or two XCDs, which would read (nearly) all of W.
struct ColumnRun { int end, c0, c1; bool near; };
HR_HD ColumnRun column_run(int t0, int t1, int tiles_m, int tiles_n) {
    const int width = kGroupM * tiles_n;
    const int group = t0 / width, first = group * width;
    const int left = tiles_m - group * kGroupM, gsz = left < kGroupM ? left : kGroupM;
    ColumnRun r;
    r.end = t1 < first + width ? t1 : first + width;
    r.c0 = (t0 - first) / gsz;
    r.c1 = (r.end - 1 - first) / gsz + 1;
    r.near = group == 0 || gsz >= kAheadShares;
    return r;
}

}  // namespace hr

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>

#include "hr_kernels.h"

namespace hr {

// The workgroups first .. end - 1 of a launch with idle CUs (wg: this one) do not take part in it: they touch the weights that the next
// launches read, XCD by XCD in the order above, 64 bytes per lane, so that those find them in their XCD's L2 (what a kernel read
// stays there for the next: 256 workgroups reading 8 MB take 1.5 us from HBM, 0.65 from their own L2 and 1.5 from
// another XCD's reading).  NW: wavefronts of a workgroup; lds: room for 256 bytes for each of them, read by nobody.
// The columns of a run are rows of W that follow each other: one run of memory.  Looked for tile by tile, at two divisions and
// ~0.2 us each, the weights of a layer took up to 24 us, longer than the attention of short documents: 0.5B shape, 16 pairs x 18 tokens,
// documents of 64 tokens 1433 -> 1113 us a call, 20 x 32 tokens 1608 -> 1451, documents of 512 tokens 1620 -> 1614.
template <int NW>
__device__ __forceinline__ void warm_weights(const WeightWalks& ws, int wg, int first, int end, char* lds) {
    typedef __attribute__((address_space(3))) void* lds_p;
    typedef const __attribute__((address_space(1))) void* gbl_p;
    const int xcd = wg % kXcds;
    const int skip = ((xcd - first) % kXcds + kXcds) % kXcds;            // first + skip: the first such workgroup on this XCD
    const int me = (wg - first - skip) / kXcds, all = (end - first - skip + kXcds - 1) / kXcds;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int i = 0; i < ws.n; ++i) {
        const WeightWalk& w = ws.w[i];
        const int n_tiles = w.tiles_m * w.tiles_n, per = (n_tiles + kXcds - 1) / kXcds;
        const int t1 = min((xcd + 1) * per, n_tiles);
        for (int t = xcd * per; t < t1;) {
            const ColumnRun r = column_run(t, t1, w.tiles_m, w.tiles_n);
            t = r.end;
            if (!r.near) continue;
            const char* base = w.W + (size_t)r.c0 * w.bn * w.row_bytes;
            const int bytes = (min(r.c1 * w.bn, w.rows) - r.c0 * w.bn) * w.row_bytes;
            for (int off = (me * NW + wave) * 4096 + lane * 64; off < bytes; off += all * NW * 4096) {
                __builtin_amdgcn_global_load_lds((gbl_p)(base + off), (lds_p)(lds + wave * 256), 4, 0, 0);
                for (int k = 0; k < ws.pace; ++k) __builtin_amdgcn_s_sleep(1);
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);              // nothing is on its way into LDS when the wave ends
}

}  // namespace hr
#endif
