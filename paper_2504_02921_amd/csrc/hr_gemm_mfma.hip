// 16-bit MFMA GEMM family for the projections of the scoring pass (gfx950).  Operands are half
// (the caller's bf16 weights are converted once when they are packed; activations are produced as half):
//   C[M][N] = A[M][K] * W[N][K]^T with fp32 accumulation and a fused epilogue
//     EPI_QKV_ROPE  : split into q / k / v, rotate-half RoPE on q and k, store half (K and V as pool-format pages)
//     EPI_RESID_ADD : x[M][N] += C   (fp32 residual stream)
//     EPI_SWIGLU    : gate/up rows interleaved in blocks of 32 -> m = silu(g) * u, store half
// Both operands are K-contiguous, which is exactly the MFMA operand order (a lane holds 8
// consecutive k of one row / column), so tiles go global -> LDS -> registers without transposes.
//
// Tiling: BM x BN x 64 macro tiles of 16 x 16 blocks of v_mfma_f32_16x16x32_f16: 256 x 256 with 8 wavefronts
// (one workgroup per CU), 320 x 256 with 8 for residual-add and long-K gate/up launches where it saves rounds of the chip,
// 128 x 128 with 4 (two per CU), wider-than-tall shapes for 128-wide heads, and ring variants with 3-18 LDS stages for
// launches of few rows; choose_gemm_launch picks per call.  LDS rows are 64 k
// (128 B) with the 16-byte chunk index XOR-swizzled by the row pair ((row >> 1) & 7): LDS serves
// 256 bytes per cycle to 16 lanes of a ds_read_b128, i.e. two 128-byte rows side by side, so 16
// consecutive rows must use 8 different chunk positions per row parity (measured: 217 B/clk/CU with
// this pattern against 119 with a (row & 7) swizzle and 32 unswizzled).
// Workgroup ids are remapped so that each XCD (ids are dealt round-robin over 8 XCDs) works on a
// contiguous run of tiles, grouped 8 tiles tall, keeping its private L2 on few A/W panels (groups 4 or 16 tall
// measured the same).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <type_traits>

#include "hr_device_types.h"
#include "hr_gemm_tiles.h"
#include "hr_internal.h"
#include "hr_kernels.h"
#include "hr_layout.h"

namespace hr {

typedef __attribute__((ext_vector_type(8))) _Float16 halfx8;
typedef __attribute__((ext_vector_type(4))) _Float16 halfx4;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(4))) unsigned uint4v;

namespace {

// What a workgroup needs first comes as parameters of its own: up to 14 words in front are in scalar registers when a wavefront starts
// (kernarg preload), where a struct's are fetched from memory.
#define HR_GEMM_PARAMS const void *A_, const void *W_, int M_, int N_, int K_, int Kw_, void *out_, const float2 *rope_, const int32_t *slot_, GemmArgs rest_
#define HR_GEMM_PASS(a) (a).A, (a).W, (int)(a).M, (a).N, (a).K, (a).Kw, EPI == EPI_RESID_ADD ? (void*)(a).x : (a).out0, (a).rope, (a).new_slot, (a)
#define HR_GEMM_WHOLE gemm_whole<EPI>(A_, W_, M_, N_, K_, Kw_, out_, rope_, slot_, rest_)
template <int EPI>
__device__ __forceinline__ GemmArgs gemm_whole(const void* A, const void* W, int M, int N, int K, int Kw, void* out, const float2* rope,
                                               const int32_t* slot, const GemmArgs& rest) {
    GemmArgs a = rest;
    a.A = A; a.W = W; a.M = M; a.N = N; a.K = K; a.Kw = Kw; a.rope = rope; a.new_slot = slot;
    if (EPI == EPI_RESID_ADD) a.x = (float*)out;
    else a.out0 = out;
    return a;
}
constexpr int BK = 64;
static_assert(kWBlock == BK, "a k-tile of W is whole lines");
constexpr int kAhead = 8, kAheadLds = 256;       // reading-ahead wavefront of the ring kernel: k-tiles, bytes of LDS
// ... and the tiles that may bring it: a smaller one asks for so little of W per k-tile that the ring is ahead enough.  Without / with
// it: 32 x 32, 65 rows, K = 4864, 10.3 / 12.3 us, but 32 x 128, 128 rows, K = 4096, 27.7 / 26.0
constexpr bool may_read_ahead(int BM, int BN, int waves) { return waves <= 4 && BM * BN >= 64 * 64; }

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* gbl_ptr_t;

// Tile loader.  The rows of a tile lie K halves apart in memory, so a lane's offset inside a pass is one 32-bit vector offset
// for all passes and k-tiles, and the rest a scalar: buffer loads straight to LDS take exactly that (no vector registers or
// additions per pass).  Rows past the end of the matrix fail the descriptor's range check; a pass without any row left
// starts at row 0 instead (its rows feed outputs that are not stored), so a scalar offset never exceeds the range.
template <int PASSES, int RPP>
struct TileSrc {
    int pass[PASSES];               // byte offset of each pass's first row
#ifdef __HIP_DEVICE_COMPILE__       // the host pass does not know the descriptor type
    __amdgpu_buffer_rsrc_t rsrc;
#endif
    __device__ __forceinline__ void set(const half_t* base, int rows, int ld) {
#ifdef __HIP_DEVICE_COMPILE__
        rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, rows * ld * 2, 0x00020000);
#endif
#pragma unroll
        for (int p = 0; p < PASSES; ++p) pass[p] = p * RPP < rows ? p * RPP * ld * 2 : 0;
    }
    __device__ __forceinline__ void load(int p, half_t* lds, int voff, int koff) const {
#ifdef __HIP_DEVICE_COMPILE__
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)lds, 16, voff, pass[p] + koff, 0, 0);
#endif
    }
};

// The same for W, from row n0 on; BLK: blocked (w_elem), a template argument so that the k loops step by constants.  N is a
// multiple of 64.  Blocked: n0 is one of 32, a pass is inside the matrix or behind it as a whole and lies in one block.  Row-major 224-column tiles start
// at multiples of 224, so that a pass may end inside the matrix and the last one of a whole tile is half beyond it: the range of `rows` rows
// in the descriptor drops those rows lane by lane, as at the end of A.
template <int BN, int RPP, bool BLK>
struct WTileSrc {
    static constexpr int PASSES = (BN + RPP - 1) / RPP;             // the last pass of a 224-row tile is half empty: out of the range
    static constexpr int kTile = (BLK ? kWBlock * BK : BK) * (int)sizeof(half_t);       // bytes from one k-tile to the next
    static __device__ __forceinline__ int row(int K) { return BLK ? kWBlock : K; }
    int pass[PASSES];
#ifdef __HIP_DEVICE_COMPILE__
    __amdgpu_buffer_rsrc_t rsrc;
#endif
    __device__ __forceinline__ void set(const half_t* W, int n0, int rows, int K) {
        constexpr bool HALF = BLK && BN < kWBlock;         // a 32-row tile may start in the middle of a block
        const int in_block = HALF ? n0 % kWBlock * kWBlock * 2 : 0;
#ifdef __HIP_DEVICE_COMPILE__
        rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (size_t)(HALF ? n0 / kWBlock * kWBlock : n0) * K), 0, (HALF ? kWBlock : rows) * K * 2, 0x00020000);
#endif
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int first = BLK ? p * RPP / kWBlock * kWBlock * K + p * RPP % kWBlock * kWBlock : p * RPP * K;
            pass[p] = (p * RPP < rows ? first * 2 : 0) + in_block;
        }
    }
    __device__ __forceinline__ void load(int p, half_t* lds, int voff, int koff) const {
#ifdef __HIP_DEVICE_COMPILE__
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)lds, 16, voff, pass[p] + koff, 0, 0);
#endif
    }
    // four bytes a lane into 256 bytes nobody reads: what counts is that their lines are in the L2 afterwards
    __device__ __forceinline__ void touch(int p, half_t* lds, int voff, int koff) const {
#ifdef __HIP_DEVICE_COMPILE__
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)lds, 4, voff, pass[p] + koff, 0, 0);
#endif
    }
};
constexpr int kNoLoad = 0x7FF00000;      // a vector offset past every range: nothing is fetched

// A thread's 16-byte chunks of the tile's part of x, for tiles whose fp32 form fits the two stages (one slab below).
template <int BN, int NT, int CHUNKS>
__device__ __forceinline__ void x_prefetch(floatx4 (&xv)[CHUNKS], const GemmArgs& a, int64_t tile_m0, int tile_n0) {
    constexpr int CPRW = BN / 4;
#pragma unroll
    for (int it = 0; it < CHUNKS; ++it) {
        const int L = it * NT + threadIdx.x, row = L / CPRW, pch = L % CPRW;
        const int64_t grow = min(tile_m0 + row, a.M - 1);
        const int col = min(tile_n0 + ((pch ^ (row & (min(CPRW, 16) - 1))) << 2), a.N - 4);
        xv[it] = *(const floatx4*)(a.x + grow * a.N + col);
    }
}

// Epilogues on transposed accumulators: a lane owns output row (lane & 15) of each 16 x 16 block and columns
// 4 * (lane >> 4) + {0..3}.  `smem` is the kernel's LDS (SA stages of A, then of W), free
// behind the main loop's last barrier except that, in a persistent launch, stage 0 may be receiving the next tile.  x_pre: what
// x_prefetch read (nullptr: x is read here).
template <int EPI, int BM, int BN, int WM, int WN, int HB, int SA>
__device__ __forceinline__ void gemm_epilogue(floatx4 (&acc)[BM / WM / 16][BN / WN / 16], const GemmArgs& a, char* smem,
                                              int64_t tile_m0, int tile_n0, const floatx4* x_pre = nullptr) {
    constexpr int NT = WM * WN * 64;
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int MI = TM / 16, NI = TN / 16;
    half_t* sA = (half_t*)smem;
    half_t* sB = sA + SA * BM * BK;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int frow = lane & 15, fq = lane >> 4;
    const int64_t row_base = tile_m0 + wm * TM + frow;
    const int col_base = tile_n0 + wn * TN + 4 * fq;
    (void)sA; (void)sB; (void)row_base; (void)col_base; (void)NT; (void)MI; (void)NI;
    if constexpr (EPI == EPI_RESID_ADD) {
        // x += C through LDS.  In the accumulator layout a lane holds 16 bytes of one row, so a direct update touches
        // 32 rows per instruction; staged as an fp32 [BM][CW] tile (16-byte chunks XOR-swizzled by the row against
        // bank conflicts of the column-wise writes) the update reads and writes whole 512-byte row segments.  The
        // stages hold BM x CW floats, so the tile goes in PASSES column slabs; a wave tile lies in one slab or is cut into
        // whole slabs.
        constexpr int LDS_BYTES = 2 * (BM + (BN + 63) / 64 * 64) * BK * (int)sizeof(half_t);
        constexpr int PASSES_MIN = (BM * BN * 4 + LDS_BYTES - 1) / LDS_BYTES;
        constexpr int PASSES = PASSES_MIN <= 2 ? PASSES_MIN : (PASSES_MIN <= 4 ? 4 : 8);     // a divisor of BN
        constexpr int CW = BN / PASSES;                 // slab width in columns
        constexpr int CPRW = CW / 4;                    // 16-byte chunks per slab row
        constexpr bool POW2 = CPRW == 8 || CPRW % 16 == 0;              // else (112-wide slabs) rows are padded instead of swizzled
        constexpr int LD = POW2 ? CW : CW + 4;
        constexpr int ITER = (BM * CPRW + NT - 1) / NT;
        // register groups of the x update (320-row tiles: 10 = 5 x 2)
        constexpr int NG = !POW2 ? (ITER + 3) / 4 : ITER == 1 ? 1 : ITER % 4 == 0 ? 4 : ITER % 5 == 0 ? 5 : 2;
        constexpr int SWZ = !POW2 ? 0 : CPRW < 16 ? CPRW - 1 : 15;
        static_assert(EPI != EPI_RESID_ADD || ((CW % TN == 0 || TN % CW == 0) && (!POW2 || (BM * CPRW) % (NG * NT) == 0) && BM * LD * 4 <= LDS_BYTES), "slab shape");
        float* stage = (float*)smem;
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            // x in NG groups of G chunks per lane (registers): the first is requested before the stage is written, so
            // its latency hides behind the write and the barrier.  Every address is clamped into the matrix, only
            // valid chunks are written back.
            constexpr int G = POW2 ? ITER / NG : 4;
            floatx4 xv[G];
            auto load_x = [&](int first) {
#pragma unroll
                for (int it = 0; it < G; ++it) {
                    const int L = (first + it) * NT + tid;
                    const int row = L / CPRW, pch = L % CPRW;
                    int col = tile_n0 + p * CW + ((pch ^ (row & SWZ)) << 2);
                    int64_t grow = tile_m0 + row;
                    grow = grow < a.M ? grow : a.M - 1;
                    col = col < a.N ? col : a.N - 4;
                    xv[it] = *(const floatx4*)(a.x + grow * a.N + col);
                }
            };
            auto update_x = [&](int first) {
#pragma unroll
                for (int it = 0; it < G; ++it) {
                    const int L = (first + it) * NT + tid;
                    const int row = L / CPRW, pch = L % CPRW;
                    const int col = tile_n0 + p * CW + ((pch ^ (row & SWZ)) << 2);
                    const int64_t grow = tile_m0 + row;
                    if (grow >= a.M || col >= a.N || (!POW2 && row >= BM)) continue;        // N is a multiple of 8: whole chunks
                    *(floatx4*)(a.x + grow * a.N + col) = xv[it] + *(const floatx4*)(stage + row * LD + (pch << 2));
                }
            };
            if (PASSES == 1 && x_pre) {
#pragma unroll
                for (int it = 0; it < G; ++it) xv[it] = x_pre[it];
            } else {
                load_x(0);
            }
            if (p > 0) __syncthreads();                 // the previous slab has been read
            constexpr int NJ = CW < TN ? CW / 16 : NI;           // blocks of a wave tile in a slab, from block j0 on
            const int j0 = CW < TN ? (p * CW % TN) / 16 : 0;
            if (CW < TN ? (p * CW) / TN == wn : (wn * TN) / CW == p) {
                const int c_off = (CW < TN ? 0 : wn * TN - p * CW) + 4 * fq;
#pragma unroll
                for (int i = 0; i < MI; ++i) {
                    const int lr = wm * TM + i * 16 + frow;
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        const int ch = (c_off + j * 16) >> 2;
                        *(floatx4*)(stage + lr * LD + ((ch ^ (lr & SWZ)) << 2)) = acc[i][j0 + j];
                    }
                }
            }
            __syncthreads();
            update_x(0);
#pragma unroll
            for (int g = 1; g < NG; ++g) {
                if (PASSES == 1 && x_pre) {
#pragma unroll
                    for (int it = 0; it < G; ++it) xv[it] = x_pre[g * G + it];
                } else {
                    load_x(g * G);
                }
                update_x(g * G);
            }
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
        static_assert(EPI != EPI_SWIGLU || NI % 4 == 0, "gate/up block pairs");
        // m = silu(g) * u goes through LDS as a half [BM][BN / 2] tile (16-byte chunks XOR-swizzled by the row) and
        // leaves in whole row segments, like the residual update above.
        constexpr int OW = BN / 2;                      // output columns of the tile
        constexpr int CPRO = OW / 8;                    // 16-byte chunks per tile row: 16 (256-byte rows) or 8 (128-byte rows)
        constexpr int ITER = BM * CPRO / NT;
        static_assert(EPI != EPI_SWIGLU || ((CPRO == 16 || CPRO == 8) && (BM * CPRO) % NT == 0), "output tile shape");
        auto swz = [](int r) { return CPRO == 16 ? (r & 15) : ((r >> 1) & 7); };
        // staged in the second stages of A and W: the first ones may already be receiving the next tile.  The tall tile's
        // output does not fit there; its launch is not persistent and stages from the start of the LDS.
        constexpr bool WHOLE = BM > 256;
        constexpr int R1 = BM * BK / OW;                 // tile rows that fit the A stage
        static_assert(EPI != EPI_SWIGLU || (WHOLE ? BM * OW <= 2 * (BM + BN) * BK : (R1 <= BM && (BM - R1) * OW <= BN * BK)),
                      "staging fits the stages");
        auto stage_row = [&](int r) {
            if constexpr (WHOLE) return (half_t*)smem + r * OW;
            else return r < R1 ? sA + BM * BK + r * OW : sB + BN * BK + (r - R1) * OW;
        };
        half_t* out = (half_t*)a.out0;
        const int F = a.N / 2;
        // split output (the layers that run with 22-bit operands): m = hi + lo is written as [M][hi F | lo F], one half
        // after the other through the same stage
        const int parts = a.split_out ? 2 : 1;
        const int ldo = parts * F;
        for (int part = 0; part < parts; ++part) {
            if (part) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");     // the hi tile has been read out of the stage
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const int lr = wm * TM + i * 16 + frow;
#pragma unroll
                for (int j = 0; j < NI; j += 4)                 // 32 gate columns, then the 32 up columns that belong to them
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const int ch = ((wn * TN) / 2 + j * 8 + b * 16) / 8 + (fq >> 1);
                        halfx4 w;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float g = acc[i][j + b][e], u = acc[i][j + 2 + b][e];
                            const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
                            const float v = g * sg * u;
                            const half_t hi = from_float<half_t>(v);
                            w[e] = part ? from_float<half_t>(v - (float)hi) : hi;
                        }
                        *(halfx4*)(stage_row(lr) + ((ch ^ swz(lr)) << 3) + 4 * (fq & 1)) = w;
                    }
            }
            // LDS-only barrier: __syncthreads() would also wait for the next tile's loads, which were just requested
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
            for (int it = 0; it < ITER; ++it) {
                const int L = it * NT + tid;
                const int row = L / CPRO, pch = L % CPRO;
                const int col = tile_n0 / 2 + ((pch ^ swz(row)) << 3);
                const int64_t grow = tile_m0 + row;
                if (grow >= a.M || col >= F) continue;          // F is a multiple of 32: whole chunks
                *(uint4v*)(out + grow * ldo + part * F + col) = *(const uint4v*)(stage_row(row) + (pch << 3));
            }
        }
    } else {   // EPI_QKV_ROPE
        constexpr int hb = 2 * HB;                              // 16-wide blocks per half head: head_dim = 64 * HB
        static_assert(EPI != EPI_QKV_ROPE || NI % (2 * hb) == 0, "a wave must hold whole heads");
        constexpr int d = 64 * HB, half = d / 2;
        const int nq = a.n_q * d, nkv = a.n_kv * d;
        // The (cos, sin) rows of this tile's tokens go to LDS first (the stages are free: nobody reads them behind
        // the last barrier of the main loop).  A lane owns one token row and would otherwise fetch its 16-byte
        // pieces of the table from 32 different cache lines per load instruction.  Chunks of 16 bytes are
        // XOR-swizzled by the row so that the 16 rows read together hit 16 different bank groups.
        constexpr int CPR = d / 4;                               // chunks per table row (d / 2 pairs of 8 bytes)
        static_assert(EPI != EPI_QKV_ROPE || (BM * CPR) % NT == 0, "table loader shape");
        static_assert(EPI != EPI_QKV_ROPE || BM * CPR * 16 <= 2 * (BM + BN) * BK * (int)sizeof(half_t), "table fits the stages");
        {
            const char* rope_bytes = (const char*)a.rope;
#pragma unroll
            for (int base = 0; base < BM * CPR; base += NT) {
                const int L = base + tid;
                const int row = L / CPR, pc = L % CPR;
                int64_t gr = tile_m0 + row;
                gr = gr < a.M ? gr : a.M - 1;
                const char* g = rope_bytes + (gr * half) * (int64_t)sizeof(float2) + ((pc ^ (row & 15)) << 4);
                __builtin_amdgcn_global_load_lds((gbl_ptr_t)g, (lds_ptr_t)(smem + (size_t)(base + wave * 64) * 16), 16, 0, 0);
            }
        }
        int slot_i[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int64_t row = row_base + i * 16;
            slot_i[i] = (a.kv_pages && row < a.M) ? a.new_slot[row] : 0;
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        // q and K quads are kept (rotated and rounded) until the table is no longer needed, then staged in LDS as a
        // half [BM][BN] tile and stored in whole row segments; V quads go straight to their pages: a wave's 16 tokens
        // fall into one or two pages, where each channel's keys are adjacent, which is as coalesced as V gets.
        halfx4 res[MI][NI];
        auto store_v_quad = [&](int i, int64_t row, int col, halfx4 w) {
            const int c_all = col - nq - nkv;
            if (!a.kv_pages) {
                *(halfx4*)((half_t*)a.out2 + row * nkv + c_all) = w;
                return;
            }
            // 16-slot pages in the pool arrangement: [page][kv head][K block | V block]
            const int kv_head = c_all / d, kv_c = c_all - kv_head * d;
            const int slot = slot_i[i];
            half_t* vb = (half_t*)a.kv_pages + ((size_t)(slot >> 4) * a.n_kv + kv_head) * (2 * kPageTokens * d) + kPageTokens * d;
            const int t = slot & 15;
#pragma unroll
            for (int e = 0; e < 4; ++e) vb[v_elem(t, kv_c + e, d)] = w[e];
        };
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int64_t row = row_base + i * 16;
            const bool row_ok = row < a.M;
            const int lrow = wm * TM + i * 16 + frow;              // row inside the tile
            const char* trow = smem + (size_t)lrow * (CPR * 16);
#pragma unroll
            for (int hbi = 0; hbi < hb; ++hbi) {
                // rotary indices hbi * 16 + 4 * fq + {0..3}: two chunks of two (cos, sin) pairs
                const int c0 = hbi * 8 + 2 * fq;
                const float4 cs01 = *(const float4*)(trow + ((c0 ^ (lrow & 15)) << 4));
                const float4 cs23 = *(const float4*)(trow + (((c0 + 1) ^ (lrow & 15)) << 4));
                const float cs_c[4] = {cs01.x, cs01.z, cs23.x, cs23.z}, cs_s[4] = {cs01.y, cs01.w, cs23.y, cs23.w};
#pragma unroll
                for (int hd = 0; hd < NI / (2 * hb); ++hd) {
                    const int jl = hd * 2 * hb + hbi, jh = jl + hb;       // low / high half of the head: same lane, same register
                    const int col_l = col_base + jl * 16, col_h = col_base + jh * 16;
                    const bool rot = col_l < nq + nkv;                      // q and k rotate, v does not
                    halfx4 wl, wh;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float lo = acc[i][jl][e], hi = acc[i][jh][e];
                        wl[e] = from_float<half_t>(rot ? rope_lo(lo, hi, cs_c[e], cs_s[e]) : lo);
                        wh[e] = from_float<half_t>(rot ? rope_hi(lo, hi, cs_c[e], cs_s[e]) : hi);
                    }
                    res[i][jl] = wl;
                    res[i][jh] = wh;
                    if (!rot && row_ok && col_l < a.N) {                  // N is a multiple of the head size
                        store_v_quad(i, row, col_l, wl);
                        store_v_quad(i, row, col_h, wh);
                    }
                }
            }
        }
        __syncthreads();                                            // every lane is done with the table
        constexpr int CPT = BN / 8;                                 // 16-byte chunks per tile row (8, 16 or 32)
        static_assert(EPI != EPI_QKV_ROPE || ((CPT == 8 || CPT % 16 == 0) && (BM * CPT) % NT == 0), "output tile shape");
        auto swz = [](int r) { return CPT == 8 ? ((r >> 1) & 7) : (r & 15); };
        half_t* stage = (half_t*)smem;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int lr = wm * TM + i * 16 + frow;
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int ch = (wn * TN + j * 16) / 8 + (fq >> 1);
                *(halfx4*)(stage + lr * BN + ((ch ^ swz(lr)) << 3) + 4 * (fq & 1)) = res[i][j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < BM * CPT / NT; ++it) {
            const int L = it * NT + tid;
            const int row = L / CPT, pch = L % CPT;
            const int col = tile_n0 + ((pch ^ swz(row)) << 3);
            const int64_t grow = tile_m0 + row;
            if (grow >= a.M || col >= nq + nkv) continue;           // past the matrix, or V (stored above)
            const uint4v w = *(const uint4v*)(stage + row * BN + (pch << 3));
            if (col < nq) {
                *(uint4v*)((half_t*)a.out0 + grow * nq + col) = w;
            } else if (!a.kv_pages) {
                *(uint4v*)((half_t*)a.out1 + grow * nkv + (col - nq)) = w;
            } else {
                const int c_all = col - nq, kv_head = c_all / d, kv_c = c_all - kv_head * d;
                const int slot = a.new_slot[grow];
                half_t* blk0 = (half_t*)a.kv_pages + ((size_t)(slot >> 4) * a.n_kv + kv_head) * (2 * kPageTokens * d);
                *(uint4v*)(blk0 + k_elem(slot & 15, kv_c, d, 2)) = w;   // 8 channels = one swizzled 16-byte chunk
            }
        }
    }
}

// BM x BN x 64 macro tile, WM x WN wavefronts, each wave (BM/WM) x (BN/WN) = MI x NI blocks of 16 x 16.
//
// What bounds it at large M is power in gate/up and at the 8B shape: with operands of full mantissas the chip holds 1.45 GHz (8B gate/up,
// K = 8192: matrix pipe busy 81 %) to 1.8 GHz (K = 896: 64 %) under this kernel, and every variant of the schedule that spends the same
// energy per product ends at the same rate.  QKV, O and down of the 0.5B shape (N = 896 and 1152; pipe busy 36-56 % at 1.84-1.90 GHz) are not at
// that limit: a tile's start, its epilogue and what the last round leaves idle.  A register-only loop reaches 1.97 PFLOP/s with v_mfma_f32_16x16x32_f16 and 1.73
// with v_mfma_f32_32x32x16_f16 (twice the accumulator traffic per product; 2.44 and 2.48 with zeros), 1.57 / 1.43 with the
// fragments read from LDS as here: hence the 16 x 16 x 32 form.
//
// Data path: buffer loads straight to LDS, 16 bytes a lane (TileSrc; nothing passes through VGPRs; lane l of a wave writes LDS bytes
// [base + 16 l, base + 16 l + 16)); SA stages of A and two of W.  A k-tile is two k-steps of 32.  A fragment of A is
// replaced by the next k-step's right behind its last MFMA, W fragments are double buffered; the k-tile's one barrier sits a
// quarter into its second k-step, when every fragment of the k-tile has been read.  Behind it the W loads of k-tile
// kt + 2 go out (their stage is free), the A loads of kt + 2 with a third stage a k-step later (a whole k-tile ahead of
// their barrier, which does not wait for them), with two stages together with W.  Requests and reads are spread over the
// MFMAs (a wave issues in order, and the CU takes 60 bytes per cycle).
// Accumulation is transposed (D = W_frag * A_frag^T): a lane owns ONE output row (lane & 15) and 4 consecutive columns
// per block, so the epilogues address one row pointer per block and store 8 / 16 bytes at a time.
template <int EPI, int BM, int BN, int WM, int WN, int HB, int SA, bool BLK>
__global__ void __launch_bounds__(WM * WN * 64, WM * WN == 4 && BM <= 128 ? 2 : 1) gemm_mfma_kernel(HR_GEMM_PARAMS) {
    GemmArgs a = HR_GEMM_WHOLE;
    constexpr int NT = WM * WN * 64;
    constexpr int TM = BM / WM, TN = BN / WN;      // wave tile
    constexpr int MI = TM / 16, NI = TN / 16;
    constexpr int RPP = NT / 8;                     // rows per loader pass (8 lanes cover one 128-byte k row)
    constexpr int PA = BM / RPP, PB = (BN + RPP - 1) / RPP, BNP = PB * RPP;
    static_assert(RPP % 16 == 0 && BM % RPP == 0 && (BN % RPP == 0 || (EPI == EPI_RESID_ADD && !BLK)), "loader shape");
    static_assert(BK == 64 && (SA == 2 || SA == 3), "two k-steps per k-tile");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    half_t* sA = (half_t*)smem;                         // [SA][BM][BK]
    half_t* sB = sA + SA * BM * BK;                     // [2][BNP][BK]

    // The gate/up launch is persistent: a workgroup walks tiles blockIdx.x, blockIdx.x + gridDim.x, ... (the same
    // XCD-chunked order) and requests the first k-tile of its next tile before it starts the epilogue of the current
    // one, so only a workgroup's first tile pays the start-up round trip (3.4k of a 50k-cycle tile at K = 896).  Its
    // epilogue has no loads that would queue behind that request.  The other launches run one tile per workgroup.
    constexpr bool PERSIST = EPI == EPI_SWIGLU && BM <= 256;
    const int tiles_m = (int)((a.M + BM - 1) / BM), tiles_n = (a.N + BN - 1) / BN;
    int vpid = blockIdx.x;
    TileCoord tc = map_tile(vpid, tiles_m, tiles_n);
    if (!tc.valid) return;
    int64_t m0;
    int n0;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int K = a.K;
    const int Kw = a.Kw > 0 ? a.Kw : K;         // columns of W: K, or K / 2 when A carries [hi | lo] halves of a split operand
    const int nkw = Kw / BK, nk = K / BK;

    // loader: lane -> LDS chunk (row lrow of the pass, physical 16-byte chunk tid & 7); it fetches the logical
    // chunk that the row-pair swizzle maps there
    const int lrow = tid >> 3;
    const int lchunk = (tid & 7) ^ ((lrow >> 1) & 7);
    const int va = (lrow * K + lchunk * 8) * 2, vb = (lrow * WTileSrc<BN, RPP, BLK>::row(Kw) + lchunk * 8) * 2;
    TileSrc<PA, RPP> srcA;
    WTileSrc<BN, RPP, BLK> srcB;
    auto set_tile = [&](const TileCoord& t) {
        m0 = (int64_t)t.tm * BM;
        n0 = t.tn * BN;
        srcA.set((const half_t*)a.A + m0 * K, (int)min((int64_t)BM, a.M - m0), K);
        srcB.set((const half_t*)a.W, n0, min(BN, a.N - n0), Kw);
    };
    set_tile(tc);
    // load p of the PA of A's k-tile kt / of the PB of W's (the LDS address is wave-uniform: the hardware adds 16 bytes per
    // lane); a k-tile past the end fetches nothing
    auto dma_a = [&](int p, int kt, int slot) {
        srcA.load(p, sA + slot * BM * BK + wave * 64 * 8 + p * NT * 8, kt < nk ? va : kNoLoad, kt < nk ? kt * (BK * 2) : 0);
    };
    auto dma_b = [&](int p, int kt, int slot) {
        const int ktw = kt < nkw ? kt : kt - nkw;             // the lo half of a split A meets the same W columns again
        srcB.load(p, sB + slot * BNP * BK + wave * 64 * 8 + p * NT * 8, kt < nk ? vb : kNoLoad, kt < nk ? ktw * srcB.kTile : 0);
    };
    auto dma_first = [&]() {                                  // k-tile 0 of a tile, into stages 0
#pragma unroll
        for (int p = 0; p < PA; ++p) dma_a(p, 0, 0);
#pragma unroll
        for (int p = 0; p < PB; ++p) dma_b(p, 0, 0);
    };

    // x of a residual add, for the tiles whose registers hold all of it: requested behind the last k-tile, one round trip instead of four in
    // the epilogue, which took half of such a tile's time.  O of the 0.5B shape (K = 896), 230 k rows 597 -> 548 us, with a third stage of
    // A 524; 65536 rows 178 -> 165 -> 158.
    constexpr bool XPRE = EPI == EPI_RESID_ADD && BM * BN <= 128 * 128;
    constexpr int XCH = BM * BN / 4 / NT;
    floatx4 xv[XPRE ? XCH : 1];
    floatx4 acc[MI][NI];
    const int frow = lane & 15, fq = lane >> 4;
    const int sw = (frow >> 1) & 7;           // row pair index: rows are 128 bytes, the bank window 256
    halfx8 af[MI], bfr[2][NI];
    // a lane's place in the first 16 rows of its wave's part of a stage, per k-step; opaque, so that the rows below fold into
    // the instruction's offset instead of a register each
    int at_a[2], at_b[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        at_a[ks] = (wm * TM + frow) * BK + (((ks * 4 + fq) ^ sw) * 8);
        at_b[ks] = (wn * TN + frow) * BK + (((ks * 4 + fq) ^ sw) * 8);
        asm("" : "+v"(at_a[ks]), "+v"(at_b[ks]));
    }
    auto read_a = [&](int i, const half_t* cA, int ks) { af[i] = *(const halfx8*)(cA + at_a[ks] + i * 16 * BK); };
    auto read_b = [&](int j, const half_t* cB, int ks) { bfr[ks][j] = *(const halfx8*)(cB + at_b[ks] + j * 16 * BK); };
    auto mfma_row = [&](int i, int ks) {
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bfr[ks][j], af[i], acc[i][j], 0, 0, 0);
    };

    using std::integral_constant;
    // how `n` operations are spread over the rows r0 .. MI - 1 of a k-step: operation q goes behind row r0 + q * (MI - r0) / n
    auto spread = [&](auto r0_c, auto n_c, int row, auto op) {
        constexpr int R0 = decltype(r0_c)::value, N = decltype(n_c)::value;
#pragma unroll
        for (int q = 0; q < N; ++q)
            if (R0 + q * (MI - R0) / N == row) op(q);
    };
    constexpr int XR = MI / 4;                 // the barrier sits behind this many rows of the second k-step
    constexpr integral_constant<int, 0> c0{};
    constexpr integral_constant<int, XR> cx{};
    constexpr integral_constant<int, PA> cpa{};
    constexpr integral_constant<int, PB> cpb{};
    constexpr integral_constant<int, NI> cni{};
    int slot_a = 0;                            // A stage of k-tile kt
    // A k-tile is a head (first k-step, the rows of the second in front of the barrier) and a tail (the barrier and the
    // rest); the loop's edge lies at the barrier, where no LDS read is outstanding.  No branch inside either; the
    // scheduling barriers keep a fragment's replacement behind the MFMAs that use it (the same registers) and the
    // memory operations spread.
    auto head = [&](int kt) {
        const half_t *cA = sA + slot_a * BM * BK, *cB = sB + (kt & 1) * BNP * BK;
        const int sa2 = slot_a == 0 ? SA - 1 : slot_a - 1;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            mfma_row(i, 0);
            __builtin_amdgcn_sched_barrier(0);
            read_a(i, cA, 1);
            spread(c0, cni, i, [&](int j) { read_b(j, cB, 1); });
            if constexpr (SA == 3) spread(c0, cpa, i, [&](int p) { dma_a(p, kt + 2, sa2); });
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < XR; ++i) mfma_row(i, 1);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto tail = [&](auto last_c, auto younger_c, int kt) {
        constexpr bool LAST = decltype(last_c)::value;
        if constexpr (!LAST) {
            // the next k-tile has landed (own loads; A of the one after, or what else was requested since, may be outstanding) and
            // every wave has read this one
            constexpr int V = (SA == 3 ? PA : 0) + decltype(younger_c)::value;
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt((V & 15) | ((V >> 4) << 14) | 0x0070);       // vmcnt(V) lgkmcnt(0)
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        const int cur = kt & 1, sa_old = slot_a;
        slot_a = slot_a + 1 == SA ? 0 : slot_a + 1;
        const half_t *nA = sA + slot_a * BM * BK, *nB = sB + (cur ^ 1) * BNP * BK;
        if constexpr (!LAST) {
#pragma unroll
            for (int r = 0; r < XR; ++r) read_a(r, nA, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = XR; i < MI; ++i) {
            mfma_row(i, 1);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!LAST) {
                read_a(i, nA, 0);
                spread(cx, cni, i, [&](int j) { read_b(j, nB, 0); });
                spread(cx, cpb, i, [&](int p) { dma_b(p, kt + 2, cur); });
                if constexpr (SA == 2) spread(cx, cpa, i, [&](int p) { dma_a(p, kt + 2, sa_old); });
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    dma_first();
    for (;;) {                                // one tile per pass; a single pass unless PERSIST
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    // k-tile 0 has landed; every wave is done with the previous tile's staging reads (PERSIST), which used the other stages
    __builtin_amdgcn_s_waitcnt(0x0F70);       // vmcnt(0)
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PB; ++p) dma_b(p, 1, 1);
#pragma unroll
    for (int p = 0; p < PA; ++p) dma_a(p, 1, 1);
    slot_a = 0;
#pragma unroll
    for (int i = 0; i < MI; ++i) read_a(i, sA, 0);
#pragma unroll
    for (int j = 0; j < NI; ++j) read_b(j, sB, 0);
    head(0);
    int kt = 0;
    for (; kt + 1 + XPRE < nk; ++kt) {
        tail(std::false_type{}, c0, kt);
        head(kt + 1);
    }
    if constexpr (XPRE) {                     // x behind the last k-tile's loads, which do not wait for it
        x_prefetch<BN, NT>(xv, a, m0, n0);
        if (kt + 1 < nk) {
            tail(std::false_type{}, integral_constant<int, XCH>{}, kt);
            head(kt + 1);
        }
    }
    tail(std::true_type{}, c0, nk - 1);
    // nobody reads the stages any more, and nothing is on its way into them
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();

    // ---- epilogue
    const int64_t tile_m0 = m0;               // the epilogue's tile; m0 / n0 move on to the next one below
    const int tile_n0 = n0;
    bool has_next = false;
    if constexpr (PERSIST) {
        vpid += (int)gridDim.x;
        const TileCoord nx = map_tile(vpid, tiles_m, tiles_n);
        has_next = nx.valid;
        if (has_next) {
            set_tile(nx);
            dma_first();                      // stages 0: nobody reads LDS behind the loop's last barrier
        }
    }
    gemm_epilogue<EPI, BM, BN, WM, WN, HB, SA>(acc, a, smem, tile_m0, tile_n0, XPRE ? xv : nullptr);
    if (!has_next) break;
    }
}

// Small-M variant: the same tile arithmetic (operand and k order as above: an output element gets the same bits from
// either) with a ring of NS LDS stages, for launches whose tiles fit the chip in about one round.  A tile then has its CU to
// itself, one wavefront per SIMD, and what counts is the serial length of a k-tile:
//   * NS k-tiles are requested ahead; vector memory operations complete in order, so "k-tile kt has landed" is a counted wait;
//   * the fragments of k-tile kt + 1 are read from LDS into a second register set before the MFMAs of k-tile kt issue, so
//     a k-tile costs one barrier (two k-tiles in deep rings), and neither LDS latency nor the loads sit in front of the matrix pipe.  The barrier that
//     says k-tile kt + 1 has landed also says that every wave holds k-tile kt in registers: its stage is free for kt + NS.
// What a k-tile takes in a full round (256 CUs, N = 4096, residual add), 64 x 64 / 160 x 64 / 128 x 128 tiles: operands in the L2s 159-177 /
// 323 / 410-450 ns; W from HBM 266 / 407 / 514, with the wavefront below 229 / 384 / 496 (16-19 TB/s into the CUs).  The same loop on
// zeros that its CU's L2 holds takes 137 / - / 284 ns, and requests alone 113 ns per 16 KiB: neither a CU's 60 bytes per cycle (16 KiB
// = 272 cycles) nor the L2s' rate to 256 CUs (35-37 TB/s) bounds a full round.  Small tiles wait for first touches of W, large ones run
// at 0.9-1.0 PFLOP/s with hot operands.  The previous loop (fragments read behind the barrier, one k-step ahead) took ~750 cycles per
// 64 x 64 k-tile whatever the number of workgroups: the down projection of 65 or 640 rows (K = 4864) 27 / 28 us.
//
// A launch of four wavefronts or fewer may bring one more (may_read_ahead, use_ahead below), which reads W kAhead k-tiles ahead of the ring and
// drops it: the tiles of one column, neighbours on one XCD, take turns, so a k-tile's lines are in their L2 when the ring asks.
// The ring alone has 128 KiB in flight: W of a 64 x 64 tile is 64 KiB of that, shared by all tiles of a column, and a first touch of
// HBM takes ~2.3 us.  Down projection of the 8B shape (K = 14336, N = 4096), 640 rows, without / with it: 139.6 / 105.1 us
// (operands in L2: 92); QKV of that shape (K = 4096), 512 rows 41.2 / 37.3.
//
// Tiles of 32 rows (32 x 32 for residual adds, 18 stages; 32 x 64 and 32 x 128 for QKV) take launches that fit one round with
// them: more k-tiles in flight, fewer bytes to deliver per k-tile and more workgroups.  65 rows, weights from HBM: down
// projection of the 0.5B shape (K = 4864) 64 x 64 17.1 -> 32 x 32 10.3 us, QKV (K = 896) 64 x 64 7.1 -> 32 x 64 5.3 us.  More rows than
// a round holds pay for A and W read twice as often: down projection, 640 rows 19.7 -> 30.5 us.
// Tiles of 96 and 160 rows x 64 (residual adds) fill rounds that the powers of two leave a third empty: 8B down projection, 640
// rows 128 x 128 (160 tiles) 105.1 -> 160 x 64 (256 tiles) 97.6 us.
template <int EPI, int BM, int BN, int WM, int WN, int HB, int NS, bool BLK>
__global__ void __launch_bounds__((WM * WN + may_read_ahead(BM, BN, WM * WN)) * 64, 1) gemm_ring_kernel(HR_GEMM_PARAMS) {
    GemmArgs a = HR_GEMM_WHOLE;
    constexpr int NT = WM * WN * 64;
    constexpr int TM = BM / WM, TN = BN / WN;
    constexpr int MI = TM / 16, NI = TN / 16;
    constexpr int RPP = NT / 8;
    constexpr int PA = BM / RPP, PB = BN / RPP;
    constexpr int KS = BK / 32;
    constexpr int LPT = PA + PB;                    // loads per thread and k-tile
    // Rings of many stages have one barrier for two k-tiles: behind it both next ones have landed, and the stages of this k-tile and the one
    // before are free, which are requested into a step later (LAG).  Whole calls, 0.5B shape, without / with: 5 candidates 973 / 965 us (32 x 32
    // tiles, 7.3 -> 7.1 us a launch), 20 candidates 1517 / 1511, 100 pairs x 4 tokens 1413 / 1404.  With six and seven stages (64 x 128 and
    // 32 x 128 tiles, W from HBM) it lost: 8B shape, 5 candidates 6090 / 6108.
    constexpr bool PAIR = NS >= 8;
    constexpr int LAG = PAIR ? 1 : 0;
    static_assert(RPP % 16 == 0 && BM % RPP == 0 && BN % RPP == 0, "loader shape");
    static_assert(NS >= 2 && (NS - 1) * LPT < 64, "the load counter has six bits");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    half_t* sA = (half_t*)smem;                         // [NS][BM][BK]
    half_t* sB = sA + NS * BM * BK;                     // [NS][BN][BK]

    const int tiles_m = (int)((a.M + BM - 1) / BM), tiles_n = (a.N + BN - 1) / BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const TileCoord tc = map_tile(blockIdx.x, tiles_m, tiles_n);
    if (!tc.valid) return;
    const int64_t m0 = (int64_t)tc.tm * BM;
    const int n0 = tc.tn * BN;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int K = a.K;
    const int Kw = a.Kw > 0 ? a.Kw : K;
    const int nkw = Kw / BK, nk = K / BK;
    TileSrc<PA, RPP> srcA;
    WTileSrc<BN, RPP, BLK> srcB;
    srcB.set((const half_t*)a.W, n0, min(BN, a.N - n0), Kw);
    if constexpr (may_read_ahead(BM, BN, WM * WN)) {
        if (wave == WM * WN) {
            if (tc.shares < kAheadShares) return;     // too few to take turns (barriers go on without the wave)
            // touches one 4-byte word of every 64 bytes: 32 rows of a k-tile per request
            WTileSrc<BN, 32, BLK> src;
            const int vt = (lane >> 1) * src.row(Kw) * 2 + (lane & 1) * 64;
            src.set((const half_t*)a.W, n0, min(BN, a.N - n0), Kw);
            int turn = NS % tc.shares;                // k-tile mod shares: whose turn it is
            auto touch = [&](int kt) {
                if (turn == tc.share && kt < nkw) {
#pragma unroll
                    for (int p = 0; p < BN / 32; ++p) src.touch(p, (half_t*)(smem + (size_t)NS * (BM + BN) * BK * sizeof(half_t)), vt, kt * src.kTile);
                }
                turn = turn + 1 == tc.shares ? 0 : turn + 1;
            };
#pragma unroll 1
            for (int kt = NS; kt < NS + kAhead; ++kt) touch(kt);
            __builtin_amdgcn_s_barrier();
#pragma unroll 1
            for (int kt = 0; kt + 1 < nk; ++kt) {     // barriers as below
                if (!PAIR || ((nk - kt) & 1) == 0) __builtin_amdgcn_s_barrier();
                touch(kt + NS + kAhead);
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);       // nothing is on its way into LDS when the wave ends
            return;
        }
    }

    // x of a residual add: requested first, so that it has arrived long before the epilogue (8B shape, 640 rows, 160 x 64 tiles: O and down
    // 69.2 -> 68.5 us on average).  A 128 x 128 tile would hold 64 registers for it through the k loop (and spilled them)
    constexpr bool XPRE = EPI == EPI_RESID_ADD && BM * BN <= 160 * 64;
    floatx4 xv[XPRE ? BM * BN / 4 / NT : 1];
    if constexpr (XPRE) x_prefetch<BN, NT>(xv, a, m0, n0);

    const int lrow = tid >> 3;
    const int lchunk = (tid & 7) ^ ((lrow >> 1) & 7);
    srcA.set((const half_t*)a.A + m0 * K, (int)min((int64_t)BM, a.M - m0), K);
    const int va = (lrow * K + lchunk * 8) * 2, vb = (lrow * srcB.row(Kw) + lchunk * 8) * 2;
    auto dma = [&](int kt, int buf) {
        half_t* da = sA + buf * BM * BK + wave * 64 * 8;
        half_t* db = sB + buf * BN * BK + wave * 64 * 8;
        const int ktw = kt < nkw ? kt : kt - nkw;
#pragma unroll
        for (int p = 0; p < PA; ++p) srcA.load(p, da + p * NT * 8, va, kt * (BK * 2));
#pragma unroll
        for (int p = 0; p < PB; ++p) srcB.load(p, db + p * NT * 8, vb, ktw * srcB.kTile);
    };
    floatx4 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int frow = lane & 15, fq = lane >> 4;
    const int a_row0 = wm * TM + frow;
    const int b_row0 = wn * TN + frow;
    const int sw = (frow >> 1) & 7;
    halfx8 af[2][KS][MI], bfr[2][KS][NI];           // fragments of a whole k-tile, double buffered
    int at_a[KS], at_b[KS];                         // as in the kernel above
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
        at_a[kk] = a_row0 * BK + (((kk * 4 + fq) ^ sw) * 8);
        at_b[kk] = b_row0 * BK + (((kk * 4 + fq) ^ sw) * 8);
        asm("" : "+v"(at_a[kk]), "+v"(at_b[kk]));
    }
    auto fload = [&](int set, int buf) {
        const half_t* cA = sA + buf * BM * BK;
        const half_t* cB = sB + buf * BN * BK;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
#pragma unroll
            for (int i = 0; i < MI; ++i) af[set][kk][i] = *(const halfx8*)(cA + at_a[kk] + i * 16 * BK);
#pragma unroll
            for (int j = 0; j < NI; ++j) bfr[set][kk][j] = *(const halfx8*)(cB + at_b[kk] + j * 16 * BK);
        }
    };

    // One k-tile, its fragments in (or on their way to) set SET, stage `slot`.  YOUNGER: how many of the k-tiles requested so
    // far come after the next one (their loads may still be outstanding), -1: there is no next one.  request: k-tile
    // kt + NS - LAG is requested into the stage that the k-tile LAG steps before leaves.
    int slot = 0;
    auto step = [&](auto set_c, auto younger_c, auto request_c, int kt) {
        constexpr int SET = decltype(set_c)::value, YOUNGER = decltype(younger_c)::value;
        constexpr bool REQUEST = decltype(request_c)::value;
        const int next = slot + 1 == NS ? 0 : slot + 1, free_slot = !PAIR ? slot : slot == 0 ? NS - 1 : slot - 1;
        if constexpr (YOUNGER >= 0 && (!PAIR || SET == 1)) {
            // the wait is the compiler's to see (its own waits in front of the MFMAs then leave the reads below alone);
            // a __syncthreads() would wait for the loads in flight as well
            constexpr int V = (YOUNGER > LAG ? YOUNGER - LAG : 0) * LPT;
            __builtin_amdgcn_s_waitcnt((V & 15) | ((V >> 4) << 14) | 0x0070);       // vmcnt(V) lgkmcnt(0)
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        // A wave issues in order, and a request or an LDS read that finds its queue full holds up the MFMAs behind it: reads and
        // requests go between the MFMAs one by one.  The order is pinned by scheduling barriers: asked for as groups, the
        // compiler kept it in one of the two copies of the loop body and put all requests in front of the MFMAs in the other.
        // Requests behind the MFMAs / spread, operands in L2, one k-tile at 2.4 GHz: 64 x 64 415 / 290 cycles, 128 x 128 945 / 593.
        constexpr int NM = KS * MI * NI, ND = KS * (MI + NI);
        const half_t *nA = sA + next * BM * BK, *nB = sB + next * BN * BK;
        half_t *dA = sA + free_slot * BM * BK + wave * 64 * 8, *dB = sB + free_slot * BN * BK + wave * 64 * 8;
        const int ktn = kt + NS - LAG, ka = ktn * (BK * 2), kb = (ktn < nkw ? ktn : ktn - nkw) * srcB.kTile;
        auto read_op = [&](int r) {
            const int rk = r / (MI + NI), f = r % (MI + NI);
            if (f < MI) af[SET ^ 1][rk][f] = *(const halfx8*)(nA + at_a[rk] + f * 16 * BK);
            else bfr[SET ^ 1][rk][f - MI] = *(const halfx8*)(nB + at_b[rk] + (f - MI) * 16 * BK);
        };
        auto request_op = [&](int p) {
            if (p < PA) srcA.load(p, dA + p * NT * 8, va, ka);
            else srcB.load(p - PA, dB + (p - PA) * NT * 8, vb, kb);
        };
        constexpr bool PIN = YOUNGER >= 0 && 2 * NM > ND;  // a 32 x 32 tile has two MFMAs: left to the groups (pinned 2.5 % slower)
        if constexpr (PIN) __builtin_amdgcn_sched_barrier(0);
        if constexpr (YOUNGER >= 0 && !PIN) {
#pragma unroll
            for (int r = 0; r < ND; ++r) read_op(r);
            if constexpr (REQUEST) {
#pragma unroll
                for (int p = 0; p < LPT; ++p) request_op(p);
            }
        }
#pragma unroll
        for (int n = 0; n < NM; ++n) {
            const int mk = n / (MI * NI), mi = n / NI % MI, mj = n % NI;
            acc[mi][mj] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bfr[SET][mk][mj], af[SET][mk][mi], acc[mi][mj], 0, 0, 0);
            if constexpr (PIN) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < ND; ++r)
                    if (r * NM / ND == n) read_op(r);
                if constexpr (REQUEST) {
#pragma unroll
                    for (int p = 0; p < LPT; ++p)
                        if (p * NM / LPT == n) request_op(p);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (YOUNGER >= 0 && !PIN) {
            constexpr int DPM = (ND + NM - 1) / NM, MD = (ND + DPM - 1) / DPM, VPM = (LPT + NM - 1) / NM, MV = (LPT + VPM - 1) / VPM;
#pragma unroll
            for (int n = 0; n < NM; ++n) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (n < MD) __builtin_amdgcn_sched_group_barrier(0x100, DPM, 0);
                if (n >= NM - MV) __builtin_amdgcn_sched_group_barrier(0x010, VPM, 0);
            }
        }
        if constexpr (YOUNGER >= 0) asm volatile("" ::: "memory");
        slot = next;
    };
    using std::integral_constant;
    constexpr int AHEAD = NS - LAG;                                 // k-tiles requested in front of the loop
    constexpr integral_constant<int, (AHEAD - 1) & 1> set_p{};      // sets alternate, counted from the last k-tile (set 0)
    constexpr integral_constant<int, AHEAD & 1> set_q{};
    constexpr integral_constant<int, AHEAD - 2> steady{};
#pragma unroll
    for (int s = 0; s < AHEAD; ++s)
        if (s < nk) dma(s, s);
    auto first_landed = [&](auto self, auto r_c) -> void {          // R k-tiles requested behind the first, of which LAG are waited for as well
        constexpr int R = decltype(r_c)::value, V = (R > LAG ? R - LAG : 0) * LPT;
        if (R == 0 || nk > R) __builtin_amdgcn_s_waitcnt((V & 15) | ((V >> 4) << 14) | 0x0F70);
        else if constexpr (R > 0) self(self, integral_constant<int, R - 1>{});
    };
    first_landed(first_landed, integral_constant<int, AHEAD - 1>{});
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if ((nk - 1) & 1) fload(1, 0);
    else fload(0, 0);
    int kt = 0;
    if (nk > AHEAD && ((nk - AHEAD) & 1)) step(set_q, steady, std::true_type{}, kt++);
    for (; kt + AHEAD < nk; kt += 2) {
        step(set_p, steady, std::true_type{}, kt);
        step(set_q, steady, std::true_type{}, kt + 1);
    }
    // the last AHEAD k-tiles (all requested): k-tile nk - 1 - R has R - 1 requested ones behind the next
    auto tail = [&](auto self, auto r_c) -> void {
        constexpr int R = decltype(r_c)::value;
        if (R < nk) step(integral_constant<int, R & 1>{}, integral_constant<int, R - 1>{}, std::false_type{}, 0);
        if constexpr (R > 0) self(self, integral_constant<int, R - 1>{});
    };
    tail(tail, integral_constant<int, AHEAD - 1>{});
    __syncthreads();                               // every wave is done reading the stages before the epilogue reuses them
    gemm_epilogue<EPI, BM, BN, WM, WN, HB, NS>(acc, a, smem, m0, n0, XPRE ? xv : nullptr);
}

int cu_count();

// Per-device "done once" flags and cached values: a host thread may drive any device, and different model handles may
// be used from different threads.
constexpr int kMaxDevices = 64;
inline int current_device() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    return dev;
}
// hipFuncSetAttribute(max dynamic LDS) once per kernel instantiation and device
template <typename K>
hipError_t allow_dynamic_lds(K kernel, size_t lds, std::atomic<uint64_t>& done) {
    const uint64_t bit = (uint64_t)1 << current_device();
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return e;
}

template <int EPI, int BM, int BN, int WM, int WN, int HB, int SA, bool BLK>
hipError_t launch_tile_of(const GemmArgs& a, hipStream_t st) {
    const int tiles_m = (int)((a.M + BM - 1) / BM), tiles_n = (a.N + BN - 1) / BN;
    const int n_tiles = tiles_m * tiles_n;
    const int per_xcd = (n_tiles + kXcds - 1) / kXcds;
    int grid = per_xcd * kXcds;
    if (EPI == EPI_SWIGLU && BM <= 256) {
        // persistent launch: as many workgroups as are resident at once (one big or two small tiles per CU), a multiple
        // of the XCD count so that the walk blockIdx.x + k * gridDim.x stays on its XCD
        const int resident = cu_count() * (BM >= 256 ? 1 : 2) / kXcds * kXcds;
        if (resident >= kXcds && grid > resident) grid = resident;
    }
    constexpr size_t lds = (size_t)(SA * BM + 2 * ((BN + 63) / 64 * 64)) * BK * sizeof(half_t);
    static std::atomic<uint64_t> attr_done{0};
    if (hipError_t e = allow_dynamic_lds(gemm_mfma_kernel<EPI, BM, BN, WM, WN, HB, SA, BLK>, lds, attr_done); e != hipSuccess) return e;
    gemm_mfma_kernel<EPI, BM, BN, WM, WN, HB, SA, BLK><<<dim3((unsigned)grid), WM * WN * 64, lds, st>>>(HR_GEMM_PASS(a));
    return hipGetLastError();
}

template <int EPI, int BM, int BN, int WM, int WN, int HB, int SA>
hipError_t launch_tile(const GemmArgs& a, const GemmPart& p, hipStream_t st) {
    if (p.bm != BM || p.bn != BN) return hipErrorInvalidValue;      // the choice and the weight walk go by the part's sizes
    if constexpr (BN == 224) {
        if (w_blocked(a.N, a.Kw > 0 ? a.Kw : a.K)) return hipErrorInvalidValue;
        return launch_tile_of<EPI, BM, BN, WM, WN, HB, SA, false>(a, st);
    } else
    return w_blocked(a.N, a.Kw > 0 ? a.Kw : a.K) ? launch_tile_of<EPI, BM, BN, WM, WN, HB, SA, true>(a, st)
                                                 : launch_tile_of<EPI, BM, BN, WM, WN, HB, SA, false>(a, st);
}

// The reading-ahead wavefront pays where several tiles share a column of W and the k loop is long.  Without / with it, weights
// from HBM, N = 4096: two row tiles of 64 lose (128 rows, K = 4096 21.0 / 23.1 us, K = 14336 70.2 / 75.6), three gain when they are
// full (192 rows 69.9 / 64.0) and lose when the last is not (145 rows 53.1 / 60.5: the short tile runs ahead of the others by
// itself), five gain (320 rows of 64 x 128, K = 4096 31.2 / 26.1, K = 14336 105.6 / 84.2); K = 2048 gains (512 rows 19.0 / 17.5), K = 896
// loses (512 rows 9.1 / 9.2, 640 rows of 64 x 64 at N = 896 5.7 / 5.8): the line lies between those two.  A rest of fewer tiles
// behind groups of eight goes without (QKV, 1034 rows of 128 x 128, K = 4096: 77 us, with it 90).
// Where the attention has read W ahead (WeightWalks) the wavefront only takes LDS and issue slots: 0.5B shape, whole calls with /
// without it: 640 tokens 1652 / 1630 us, 1000 1963 / 1949, 2000 2879 / 2842, 4000 4283 / 4274.
inline bool use_ahead(const GemmArgs& a, int tiles_m) { return !a.w_near && tiles_m >= kAheadShares && a.K >= 2048; }

template <int EPI, int BM, int BN, int WM, int WN, int HB, int NS, bool BLK>
hipError_t launch_ring_of(const GemmArgs& a, hipStream_t st) {
    const int tiles_m = (int)((a.M + BM - 1) / BM), tiles_n = (a.N + BN - 1) / BN;
    const int grid = (tiles_m * tiles_n + kXcds - 1) / kXcds * kXcds;
    constexpr bool may = may_read_ahead(BM, BN, WM * WN);
    const bool ahead = may && use_ahead(a, tiles_m);
    constexpr size_t ring = (size_t)NS * (BM + BN) * BK * sizeof(half_t), lds_most = ring + (may ? kAheadLds : 0);
    static std::atomic<uint64_t> attr_done{0};
    if (hipError_t e = allow_dynamic_lds(gemm_ring_kernel<EPI, BM, BN, WM, WN, HB, NS, BLK>, lds_most, attr_done); e != hipSuccess) return e;
    gemm_ring_kernel<EPI, BM, BN, WM, WN, HB, NS, BLK><<<dim3((unsigned)grid), (WM * WN + ahead) * 64, ahead ? lds_most : ring, st>>>(HR_GEMM_PASS(a));
    return hipGetLastError();
}

template <int EPI, int BM, int BN, int WM, int WN, int HB, int NS>
hipError_t launch_ring(const GemmArgs& a, const GemmPart& p, hipStream_t st) {
    if (p.bm != BM || p.bn != BN) return hipErrorInvalidValue;      // the choice and the weight walk go by the part's sizes
    return w_blocked(a.N, a.Kw > 0 ? a.Kw : a.K) ? launch_ring_of<EPI, BM, BN, WM, WN, HB, NS, true>(a, st)
                                                 : launch_ring_of<EPI, BM, BN, WM, WN, HB, NS, false>(a, st);
}

int cu_count() {
    static std::atomic<int> cache[kMaxDevices];
    const int dev = current_device();
    int n = cache[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cache[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

}  // namespace

int device_cu_count() { return cu_count(); }

bool gemm_mfma_supported(const hr_model_cfg& c) {
    if (c.dtype != HR_BF16) return false;
    if (c.head_dim != 64 && c.head_dim != 128) return false;
    const int nq = c.n_q_heads * c.head_dim;
    if (c.hidden % BK != 0 || c.ffn % BK != 0 || nq % BK != 0) return false;   // every K is a multiple of 64
    if (c.ffn % 32 != 0) return false;                                         // gate/up interleave of 32
    return true;
}

// the same launch for the rows behind the first `rows`
static void advance_rows(GemmEpilogue epi, GemmArgs& r, int64_t rows) {
    auto halves = [&](void* p, int64_t per_row) { return p ? (void*)((half_t*)p + rows * per_row) : nullptr; };
    r.A = (const half_t*)r.A + rows * r.K;
    if (epi == EPI_RESID_ADD) r.x += rows * r.N;
    if (epi == EPI_SWIGLU) r.out0 = halves(r.out0, (r.split_out ? 2 : 1) * (int64_t)(r.N / 2));
    if (epi == EPI_QKV_ROPE) {
        r.out0 = halves(r.out0, (int64_t)r.n_q * r.d);
        if (!r.kv_pages) {                      // with pages the slots say where K and V go
            r.out1 = halves(r.out1, (int64_t)r.n_kv * r.d);
            r.out2 = halves(r.out2, (int64_t)r.n_kv * r.d);
        }
        r.rope += rows * (r.d / 2);
        if (r.new_slot) r.new_slot += rows;
    }
}

static GemmKind kind_of(GemmEpilogue epi, const GemmArgs& a) {
    const bool wide_head = epi == EPI_QKV_ROPE && a.d == 128;       // a wave must span a whole 128-wide head
    return epi == EPI_RESID_ADD ? GEMM_RESID : epi == EPI_SWIGLU ? GEMM_SWIGLU : wide_head ? GEMM_QKV128 : GEMM_QKV64;
}

// The XCDs' L2s hold 4 MiB each; the activations pass through them as well.  A layer of the 0.5B shape is 28.4 MiB.  O alone of the
// 8B shape (32 MiB): 100 rows 6083 -> 5946 us a call, 640 rows 10630 -> 10680.
// Matrices that are left out do not count, although their bytes pass through the L2s in between: 16 layers of hidden 2048 and ffn 8192 (gate / up
// and down, 96 MiB, left out), nothing / O / O and QKV read ahead, 1300 rows 3635 / 3630 / 3600 us a call (640 rows 2173 each); 28 layers of
// 1536 and 8960, 160 rows 2585 / 2563 / 2490.
constexpr int64_t kWarmBytes = (int64_t)30 << 20;

bool gemm_weight_walk(GemmEpilogue epi, const GemmArgs& a, WeightWalks* out) {
    const GemmKind kind = kind_of(epi, a);
    const GemmLaunch g = choose_gemm_launch(kind, a.M, a.N, a.K, cu_count(), a.beside);
    const int Kw = a.Kw > 0 ? a.Kw : a.K;
    const int64_t bytes = (int64_t)a.N * Kw * (int64_t)sizeof(half_t);
    if (g.n != 1 || out->n >= kWarmMost || out->bytes + bytes > kWarmBytes) return false;
    const int bm = g.part[0].bm;
    int bn = g.part[0].bn;
    if (w_blocked(a.N, Kw)) bn = std::max(bn, kWBlock);       // what is walked is one run of memory: whole blocks
    WeightWalk& w = out->w[out->n++];
    w.W = (const char*)a.W;
    w.row_bytes = Kw * (int)sizeof(half_t);
    w.rows = a.N;
    w.tiles_m = (int)((a.M + bm - 1) / bm);
    w.tiles_n = (a.N + bn - 1) / bn;
    w.bn = bn;
    out->bytes += bytes;
    return true;
}

hipError_t launch_gemm_mfma(GemmEpilogue epi, const GemmArgs& a, hipStream_t st) {
    if (a.M == 0) return hipSuccess;
    if (a.K % BK != 0) return hipErrorInvalidValue;
    if (a.Kw > 0 && (a.Kw % BK != 0 || (a.K != a.Kw && a.K != 2 * a.Kw))) return hipErrorInvalidValue;
    const GemmKind kind = kind_of(epi, a);
    const GemmLaunch g = choose_gemm_launch(kind, a.M, a.N, a.K, cu_count(), a.beside);
    GemmArgs r = a;
    for (int i = 0; i < g.n; ++i) {
        const GemmPart& p = g.part[i];
        r.M = p.rows;
        hipError_t e = hipErrorInvalidValue;
        switch (kind) {
            case GEMM_QKV64:
                switch (p.tile) {
                    case GT_BIG: e = launch_tile<EPI_QKV_ROPE, 256, 256, 2, 4, 1, 3>(r, p, st); break;
                    case GT_SMALL: e = launch_tile<EPI_QKV_ROPE, 128, 128, 2, 2, 1, 3>(r, p, st); break;
                    case GT_RING128: e = launch_ring<EPI_QKV_ROPE, 128, 128, 2, 2, 1, 4>(r, p, st); break;
                    case GT_RING64: e = launch_ring<EPI_QKV_ROPE, 64, 64, 2, 1, 1, 8>(r, p, st); break;
                    case GT_RING32_64: e = launch_ring<EPI_QKV_ROPE, 32, 64, 2, 1, 1, 8>(r, p, st); break;
                    default: break;
                }
                break;
            case GEMM_QKV128:
                switch (p.tile) {
                    case GT_BIG: e = launch_tile<EPI_QKV_ROPE, 256, 256, 4, 2, 2, 3>(r, p, st); break;
                    case GT_RING128: e = launch_ring<EPI_QKV_ROPE, 128, 128, 4, 1, 2, 4>(r, p, st); break;
                    case GT_RING64_128: e = launch_ring<EPI_QKV_ROPE, 64, 128, 4, 1, 2, 6>(r, p, st); break;
                    case GT_RING32_128: e = launch_ring<EPI_QKV_ROPE, 32, 128, 2, 1, 2, 7>(r, p, st); break;
                    default: break;
                }
                break;
            case GEMM_RESID:
                switch (p.tile) {
                    case GT_BIG:
                        e = p.bn == 224 ? launch_tile<EPI_RESID_ADD, 256, 224, 4, 2, 1, 3>(r, p, st) : launch_tile<EPI_RESID_ADD, 256, 256, 2, 4, 1, 3>(r, p, st);
                        break;
                    case GT_TALL: e = launch_tile<EPI_RESID_ADD, 320, 256, 2, 4, 1, 2>(r, p, st); break;
                    case GT_SMALL: e = launch_tile<EPI_RESID_ADD, 128, 128, 2, 2, 1, 3>(r, p, st); break;
                    case GT_RING128: e = launch_ring<EPI_RESID_ADD, 128, 128, 2, 2, 1, 4>(r, p, st); break;
                    case GT_RING64_128: e = launch_ring<EPI_RESID_ADD, 64, 128, 2, 2, 1, 6>(r, p, st); break;
                    case GT_RING160_64: e = launch_ring<EPI_RESID_ADD, 160, 64, 2, 2, 1, 5>(r, p, st); break;
                    case GT_RING96_64: e = launch_ring<EPI_RESID_ADD, 96, 64, 2, 2, 1, 7>(r, p, st); break;
                    case GT_RING64: e = launch_ring<EPI_RESID_ADD, 64, 64, 2, 2, 1, 9>(r, p, st); break;
                    case GT_RING32: e = launch_ring<EPI_RESID_ADD, 32, 32, 2, 2, 1, 18>(r, p, st); break;
                    default: break;
                }
                break;
            case GEMM_SWIGLU:
                switch (p.tile) {
                    case GT_BIG: e = launch_tile<EPI_SWIGLU, 256, 256, 2, 4, 1, 3>(r, p, st); break;
                    case GT_TALL: e = launch_tile<EPI_SWIGLU, 320, 256, 2, 4, 1, 2>(r, p, st); break;
                    case GT_SMALL: e = launch_tile<EPI_SWIGLU, 128, 128, 2, 2, 1, 2>(r, p, st); break;
                    case GT_RING128_256: e = launch_ring<EPI_SWIGLU, 128, 256, 2, 4, 1, 3>(r, p, st); break;
                    case GT_RING128: e = launch_ring<EPI_SWIGLU, 128, 128, 2, 2, 1, 4>(r, p, st); break;
                    case GT_RING64_128: e = launch_ring<EPI_SWIGLU, 64, 128, 2, 2, 1, 6>(r, p, st); break;
                    default: break;
                }
                break;
        }
        if (e != hipSuccess) return e;
        if (i + 1 < g.n) advance_rows(epi, r, p.rows);
    }
    return hipSuccess;
}

}  // namespace hr
