// In-page arrangement of the document-KV pool (private to the library), shared by the kernel that
// writes pages and the kernels that read them.  Offsets are in elements of the pool dtype.
//
// A page holds 16 tokens of one (layer, kv head): a K block followed by a V block, 16 * d elements
// each, so one page is a single contiguous burst (4 KiB at d = 64, 8 KiB at d = 128 for 16-bit KV).
//   K block: token-major rows of d channels with the 8-channel chunk index XOR-swizzled by the token
//            index.  The swizzle is the LDS bank pattern the MFMA fragment reads want (LDS has 64 banks
//            of 4 bytes = 256 bytes per cycle, and a 16-byte read serves 16 lanes per cycle, so the 16
//            rows read together must land on 16 different 16-byte positions of that 256-byte window:
//            128-byte rows are swizzled by the row pair (t >> 1) & 7, 256-byte rows by t & 15).  It is
//            baked into HBM so that a page is copied to LDS verbatim.
//   V block: transposed and split by key parity group: [t bit 2][channel][8 keys], where the 8 keys
//            of a group are t = {0,1,2,3,8,9,10,11} (+4 for the second group).  A wavefront lane that
//            feeds v_mfma_f32_32x32x16 with V^T reads its 8 keys as one 16-byte word.
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#define HR_HD __host__ __device__ inline __attribute__((always_inline))
#else
#define HR_HD inline
#endif

namespace hr {

// esz: bytes per element of the pool dtype
HR_HD int k_swizzle(int t, int d, int esz) {
    if (esz > 2) return 0;                       // fp32 pages are read straight into registers, not through LDS
    const int row_bytes = d * esz;
    return row_bytes == 128 ? ((t >> 1) & 7) : row_bytes == 256 ? (t & 15) : 0;
}

HR_HD int k_elem(int t, int c, int d, int esz) { return t * d + ((((c >> 3) ^ k_swizzle(t, d, esz)) << 3) | (c & 7)); }

HR_HD int v_elem(int t, int c, int d) { return ((t >> 2) & 1) * (d * 8) + c * 8 + ((t & 3) | ((t & 8) >> 1)); }

// Packed 16-bit weights [N][K] (N, K multiples of 64).  Large matrices are kept in blocks of 64 rows, in a block k-tile after
// k-tile of [64 rows][64 k]: what a 64-row tile reads per k-tile is 8 KiB in one piece and follows the k-tile before, where
// rows K apart are 64 places in memory.  8B shape (H = 4096, weights from HBM), whole calls row-major / blocked: 60 tokens
// 5147 / 4856 us, 100 tokens 6070 / 5638, 250 tokens 6850 / 6542, 400 tokens 8855 / 8580, 10k tokens 146.7 / 145.3 ms.
// Matrices that are narrow or short stay row-major: with those of the 0.5B shape (N or K of 896) blocked, whose 32-row tiles read
// half blocks, a call of 150 tokens took 1112 us against 1104.
constexpr int kWBlock = 64, kWBlockMin = 2048;       // rows of a block; the least N and K of a matrix kept in blocks
HR_HD bool w_blocked(int N, int K) { return N >= kWBlockMin && K >= kWBlockMin; }
HR_HD int64_t w_elem(int64_t n, int k, int N, int K) {
    if (!w_blocked(N, K)) return n * K + k;
    return n / kWBlock * kWBlock * K + (int64_t)(k / kWBlock) * (kWBlock * kWBlock) + n % kWBlock * kWBlock + k % kWBlock;
}

}  // namespace hr
