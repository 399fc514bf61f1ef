// Paged grouped-query prefix attention for launches of few query rows (gfx950): the same values as hr_attn_mfma.hip, bit for
// bit, with a work item's keys spread over wavefronts.
//
// There a wavefront walks the keys of its 32 query rows in one chain (S -> maximum -> exp -> P -> O per 32 keys), which fills
// the chip when there are many rows; a request of a few candidates has 30 to 600 blocks of 32 rows for 1024 SIMDs, and its launch
// lasts as long as one chain.  Only two things in that chain depend on the keys before: the running maximum, a few scalar steps per
// row, and the order of the sums in O.  So here a workgroup takes one block of 32 rows of one (pair, kv head), and
//   * kSWaves wavefronts compute S and its row maxima for every kSWaves-th sub-tile of 32 keys, all of them independent;
//   * behind a barrier each walks the maxima in key order (the same lazily moved maximum as there) and turns its S into P;
//   * behind another barrier kOWaves wavefronts, each with channels of its own, add V P to O in key order.  Their V, and the
//     first K, is requested before anything else; O of one round is added while S of the next is computed.
// K goes to the wavefront that uses it: whole lines into registers, then through LDS into MFMA order (in that order from memory each
// 16-byte piece of a load would be a line of its own).  The blocks of a (pair, kv head) run on one XCD, whose L2 serves all
// of them but the first.
//
// Measured, one launch: 0.5B shape, 30 blocks of 100-300 keys 14.4 -> 10 us, 40 blocks (last layer) of 544 keys 15.2 -> 13 us, 280 blocks of 544
// keys, with the layer's weights read ahead beside them, 17.1 -> 14.5 us.  What is left, in cycles of 2.4 GHz and one workgroup of 10
// sub-tiles (18 k): 3 k from its start to the page ids' request, 0.8 k for the ids, 5.5 k until the first K is there (pages of a
// layer that no TLB has seen: up to 10 k), 2 k for S of two sub-tiles, 2.5 k for their P, 2.7 k for V P, 1 k for the output.
// Tried and not kept: eight wavefronts' S of three sub-tiles each in one round (spills at two workgroups per CU); page ids as scalars per
// sub-tile (64-bit products in the scalar unit: 50 instructions a sub-tile); the pages touched by the idle CUs of the QKV launch in front
// (attention 10.1 -> 9.1 us, gate / up 7.2 -> 7.8, the call 1004 -> 1000).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>

#include "hr_attn_common.h"
#include "hr_attn_rows.h"
#include "hr_device_types.h"
#include "hr_gemm_tiles.h"
#include "hr_internal.h"
#include "hr_kernels.h"
#include "hr_layout.h"

namespace hr {

namespace {

typedef __attribute__((ext_vector_type(4))) unsigned uint4v;
typedef const __attribute__((address_space(1))) char* gbl_char_t;      // without it a pointer made of two words is loaded from as flat memory
typedef const __attribute__((address_space(1))) uint4v* gbl_word_t;
struct __attribute__((packed, aligned(8))) Word8 { uint4v w; };
typedef const __attribute__((address_space(1))) Word8* gbl_word8_t;

constexpr int kWaves = kRowsWaves;

template <int HD>
struct RowsGeo {
    static constexpr int NSUB = kRoundSubs, V_AHEAD = kVAhead;
    static constexpr int MBW = HD / 32 / kOWaves;            // 32-channel blocks per O wavefront
    static constexpr int KB = kPageTokens * HD * 2;          // bytes of a half page's K (or V) block
    // LDS: P, each S wavefront's K in page order, row maxima (two rounds), row sums, rescaling factors, 256 bytes that nobody reads
    static constexpr int P_AT = 0, K_AT = P_AT + NSUB * 2048, MX_AT = K_AT + kSWaves * 2 * KB, SUM_AT = MX_AT + 2 * NSUB * 128,
                         ALPHA_AT = SUM_AT + NSUB * 256, TOUCH_AT = ALPHA_AT + NSUB * 128,
                         LDS = TOUCH_AT + kSWaves * 256;
};

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }      // loads stay in flight

// What a workgroup divides by comes with a multiplier (exact for dividend x divisor below 2^32): a division is 40 instructions
inline unsigned make_divisor(int n) { return n > 1 ? (unsigned)((((uint64_t)1 << 32) + n - 1) / n) : 0u; }
__device__ __forceinline__ int divided(int a, unsigned mul) { return mul ? (int)__umulhi((unsigned)a, mul) : a; }

// The first 14 words of the parameters are in scalar registers when a wavefront starts (kernarg preload): what it needs to find its
// pages.  shape: see rows_holds.
template <int HD, bool FP8>
__global__ void __launch_bounds__(kWaves * 64) __attribute__((amdgpu_waves_per_eu(HD == 64 ? 4 : 2, 8))) attn_rows_kernel(
    const int32_t* __restrict__ m_cu, const int32_t* __restrict__ m_prefix, const int32_t* __restrict__ m_pt, const int32_t* __restrict__ m_new_cu,
    int pt_stride, int n_kv, unsigned mul_kv, int g, unsigned mul_g, unsigned shape, const half_t* __restrict__ q, const char* __restrict__ kv_new,
    half_t* __restrict__ o, const char* __restrict__ layer_data, const float* __restrict__ layer_scales, int warm_wgs, WeightWalks warm) {
    using G = RowsGeo<HD>;
    constexpr int KC = HD / 16, KB = G::KB, PAGE = 2 * KB;                        // half pages
    constexpr int KBP = FP8 ? KB / 2 : KB, PAGE_P = 2 * KBP;                      // the pool's
    constexpr int KL = 2 * KB / 1024;                                             // 16-byte loads per lane and sub-tile
    constexpr int NSUB = G::NSUB;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int blocks = shape >> 1 & 0xFF, n_seq = shape >> 9;
    const bool last_only = shape & 1;
    if ((int)blockIdx.y >= blocks) {                                              // behind the rows' workgroups
        const int first = blocks * (int)gridDim.x, me = (int)(blockIdx.y * gridDim.x + blockIdx.x);
        if (me < first + warm_wgs) warm_weights<kWaves>(warm, me, first, first + warm_wgs, smem);
        return;
    }
    const int row0 = (int)blockIdx.y * 32;
    const int p = divided((int)blockIdx.x, mul_kv), h = (int)blockIdx.x - p * n_kv;
    if (p >= n_seq) return;
    const int t0 = m_cu[p], qn = m_cu[p + 1] - t0, D = m_prefix[p], own_page = m_new_cu[p] >> 4;
    const int M = last_only ? g : qn * g;
    if (row0 >= M) return;
    const int lane = threadIdx.x & 63, ln = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_doc = (D + 31) / 32;                                              // sub-tiles of the document
    const int n_sub = n_doc + (last_only ? qn - 1 : divided(min(row0 + 31, M - 1), mul_g)) / 32 + 1;   // ... and of the own keys that some row sees
    const int last_page = (D + kPageTokens - 1) / kPageTokens - 1;
    const int32_t* pt = last_page >= 0 ? m_pt + (size_t)p * pt_stride : m_cu;     // no document: read and not used
    const int row = row0 + ln, rc = min(row, M - 1);
    const int row_i = last_only ? qn - 1 : divided(rc, mul_g), head = last_only ? rc : rc - row_i * g;
    const float c_log2 = 1.4426950408889634f / sqrtf((float)HD);
    float* s_max = (float*)(smem + G::MX_AT);                                     // [2][NSUB][32]
    float* s_sum = (float*)(smem + G::SUM_AT);                                    // [NSUB][64]
    float* s_alpha = (float*)(smem + G::ALPHA_AT);                                // [NSUB][32]

    // lane l has the address (and the fp8 scales) of page l of two rounds: a document's pages, past the end the last one again
    // (finite data, masked), then the own keys'; behind the last sub-tile that one's again
    struct Pages { uint64_t at; float sk, sv; };
    auto load_pages = [&](int round) {                                            // an even one
        const int jj = rows_lane_sub(round, lane, n_sub), side = lane & 1;
        const unsigned id = pt[max(min(2 * jj + side, last_page), 0)];
        const uint64_t doc = (uint64_t)id * (unsigned)(n_kv * PAGE_P) + (uint64_t)(layer_data + h * PAGE_P);
        const uint64_t own = (uint64_t)(unsigned)(own_page + (jj - n_doc) * 2 + side) * (unsigned)(n_kv * PAGE) + (uint64_t)(kv_new + h * PAGE);
        Pages r;
        r.at = jj < n_doc ? doc : own;
        if constexpr (FP8) {
            const float2 s = *(const float2*)(layer_scales + ((size_t)(jj < n_doc ? id : 0) * n_kv + h) * 2);
            r.sk = s.x;
            r.sv = s.y;
        }
        return r;
    };
    auto page_at = [&](const Pages& pg, int l) {
        const unsigned lo = __builtin_amdgcn_readlane((unsigned)pg.at, l), hi = __builtin_amdgcn_readlane((unsigned)(pg.at >> 32), l);
        return (gbl_char_t)((uint64_t)hi << 32 | lo);
    };
    // to the next pair of rounds: a branch of its own, or the compiler would select among registers and wait for `b` in every round
    auto follow = [](Pages& a, const Pages& b) {
        a = b;
        asm volatile("" : "+v"(a.at));
    };
    auto lane_of = [](float v, int l) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), l)); };
    const int rounds = (n_sub + NSUB - 1) / NSUB;
    Pages cur = load_pages(0);

    // Every load below is made whether its sub-tile exists or not: behind a branch the compiler could not count the loads that are younger
    // than the one it waits for, and would wait for all of them.
    if (wave < kSWaves) {
        const half_t* qr = q + ((size_t)(t0 + row_i) * n_kv * g + h * g + head) * HD;
        halfx8 qf[KC];
#pragma unroll
        for (int kk = 0; kk < KC; ++kk) qf[kk] = *(const halfx8*)(qr + (2 * kk + hh) * 8);
        char* kbuf = smem + G::K_AT + wave * 2 * KB;
        uint4v kr[kSPW][KL];
        auto load_k = [&](const Pages& pg, int round, int i) {                    // the wave's i-th sub-tile of the round
            const int j = wave + kSWaves * i;
            const gbl_char_t a = page_at(pg, rows_page_lane(round, j, 0)), b = page_at(pg, rows_page_lane(round, j, 1));
            const bool doc8 = FP8 && round * NSUB + j < n_doc;                    // half as many bytes: read twice
#pragma unroll
            for (int e = 0; e < KL; ++e) {
                if (doc8) kr[i][e] = *(gbl_word_t)((e / (KL / 4) % 2 ? b : a) + e % (KL / 4) * 1024 + lane * 16);
                else kr[i][e] = *(gbl_word_t)((e < KL / 2 ? a : b) + e % (KL / 2) * 1024 + lane * 16);
            }
            // four bytes of every line of V into LDS that nobody reads: the O wavefronts' requests then find it in the L2
            const int vb = doc8 ? KBP : KB;
            __builtin_amdgcn_global_load_lds((gbl_ptr_t)((hh ? b : a) + vb + ln * (vb / 32)), (lds_ptr_t)(smem + G::TOUCH_AT + wave * 256), 4, 0, 0);
        };
#pragma unroll
        for (int i = 0; i < kSPW; ++i) load_k(cur, 0, i);
        float m_run = -INFINITY;
        Pages ahead = cur, nxt = cur;
        for (int r = 0; r < rounds; ++r) {
            const int j0 = r * NSUB;
            const int l0 = (r & 1) * 2 * NSUB;                                    // the round's first page among the lanes
            floatx16 s[kSPW];
            float cs[kSPW][2];
            float* mx_out = s_max + (r & 1) * NSUB * 32;
#pragma unroll
            for (int i = 0; i < kSPW; ++i) {
                const int j = wave + kSWaves * i;
                const bool doc8 = FP8 && j0 + j < n_doc;
                const int t = ln & 15;
                halfx8 kf[KC];
                __builtin_amdgcn_wave_barrier();           // LDS accesses of one wave execute in order: the previous sub-tile has been read
#pragma unroll
                for (int e = 0; e < KL; ++e) *(uint4v*)(kbuf + e * 1024 + lane * 16) = kr[i][e];
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int kk = 0; kk < KC; ++kk) {
                    if (doc8)
                        kf[kk] = fp8x8_to_half(*(const uint2*)(kbuf + (ln >> 4) * KBP + t * HD + (((2 * kk + hh) ^ k_swizzle(t, HD, 1)) << 3)),
                                               fp8_expand_factor(1.0f));
                    else
                        kf[kk] = *(const halfx8*)(kbuf + (ln >> 4) * KB + (t * HD + (((2 * kk + hh) ^ k_swizzle(t, HD, 2)) << 3)) * 2);
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) s[i][e] = 0.f;
#pragma unroll
                for (int kk = 0; kk < KC; ++kk) s[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[kk], qf[kk], s[i], 0, 0, 0);
                cs[i][0] = c_log2;
                cs[i][1] = c_log2;
                if (doc8) {
                    cs[i][0] *= lane_of(cur.sk, l0 + 2 * j);
                    cs[i][1] *= lane_of(cur.sk, l0 + 2 * j + 1);
                }
            }
#pragma unroll
            for (int i = 0; i < kSPW; ++i) {
                const int j = wave + kSWaves * i;
                const bool doc = j0 + j < n_doc;
                // a lane holds keys 8 * (e >> 2) + 4 * hh + (e & 3) of the sub-tile for query row ln; keys [0, limit) are visible
                const int key0 = 32 * (j0 + j - n_doc);
                if (!doc || D - 32 * (j0 + j) < 32) {
                    const int limit = (doc ? D - 32 * (j0 + j) : j0 + j < n_sub ? min(qn - key0, row_i + 1 - key0) : 0) - 4 * hh;
#pragma unroll
                    for (int e = 0; e < 16; ++e) s[i][e] = 8 * (e >> 2) + (e & 3) < limit ? s[i][e] : -INFINITY;
                }
                float mx0 = s[i][0], mx1 = s[i][8];
#pragma unroll
                for (int e = 1; e < 8; ++e) {
                    mx0 = fmaxf(mx0, s[i][e]);
                    mx1 = fmaxf(mx1, s[i][8 + e]);
                }
                mx_out[j * 32 + ln] = row_max2(fmaxf(mx0 * cs[i][0], mx1 * cs[i][1]));     // of an absent sub-tile: nothing visible
            }
            if (r & 1) follow(ahead, nxt);
#pragma unroll
            for (int i = 0; i < kSPW; ++i) load_k(ahead, rows_asked(r + 1, rounds), i);
            if (rows_fetches_pages(r, rounds)) nxt = load_pages(r + 2);
            asm volatile("" ::: "memory");
            lds_barrier();                                                        // the maxima are there; P has been read
            // The running maximum in front of and behind the wave's sub-tiles; it only follows scores that exceed it by more than kLazyMax
            float mb[kSPW], mh[kSPW];
#pragma unroll
            for (int i = 0; i < kSPW; ++i) {
                float mx[kSWaves];
#pragma unroll
                for (int w = 0; w < kSWaves; ++w) mx[w] = mx_out[(i * kSWaves + w) * 32 + ln];
#pragma unroll
                for (int w = 0; w < kSWaves; ++w) {
                    const float c = fmaxf(m_run, mx[w]), m = c > m_run + kLazyMax ? c : m_run;
                    mb[i] = w == 0 || wave == w ? m_run : mb[i];
                    mh[i] = w == 0 || wave == w ? m : mh[i];
                    m_run = m;
                }
            }
#pragma unroll
            for (int i = 0; i < kSPW; ++i) {
                const int j = wave + kSWaves * i;
                const float m_use = mh[i] == -INFINITY ? 0.f : mh[i];             // a row with nothing visible yet keeps p = 0
                s_alpha[j * 32 + ln] = mb[i] == mh[i] ? 1.0f : mb[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mb[i] - mh[i]);
                float vs0 = 1.f, vs1 = 1.f;
                if (FP8 && j0 + j < n_doc) {
                    vs0 = fp8_scale_mantissa(lane_of(cur.sv, l0 + 2 * j));
                    vs1 = fp8_scale_mantissa(lane_of(cur.sv, l0 + 2 * j + 1));
                }
                float lsum = 0.f;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float pr = __builtin_amdgcn_exp2f(fmaf(s[i][e], cs[i][e < 8 ? 0 : 1], -m_use));
                    lsum += pr;
                    s[i][e] = pr;
                }
                halfx8 pf[2];
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const floatx2 a = {FP8 ? s[i][e] * vs0 : s[i][e], FP8 ? s[i][e + 1] * vs0 : s[i][e + 1]};
                    const floatx2 b = {FP8 ? s[i][8 + e] * vs1 : s[i][8 + e], FP8 ? s[i][9 + e] * vs1 : s[i][9 + e]};
                    const halfx2 ha = __builtin_convertvector(a, halfx2), hb = __builtin_convertvector(b, halfx2);
                    pf[0][e] = ha[0]; pf[0][e + 1] = ha[1];
                    pf[1][e] = hb[0]; pf[1][e + 1] = hb[1];
                }
                s_sum[j * 64 + lane] = lsum;
                *(halfx8*)(smem + G::P_AT + j * 2048 + lane * 16) = pf[0];
                *(halfx8*)(smem + G::P_AT + j * 2048 + 1024 + lane * 16) = pf[1];
            }
            lds_barrier();                                                        // P is there
            if (FP8 && (r & 1)) cur = ahead;
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);          // nothing is on its way into LDS when the wave ends
        return;
    }
    const int ch0 = (wave - kSWaves) * G::MBW * 32;                               // this wave's first channel
    floatx16 oacc[G::MBW];
#pragma unroll
    for (int mb = 0; mb < G::MBW; ++mb)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[mb][e] = 0.f;
    float l_run = 0.f;
    uint4v vr[G::V_AHEAD][G::MBW][2];                // fp8: the first half of each counts; the last channel's ends 8 bytes behind its page
    auto load_v = [&](const Pages& pg, int round, int j) {
        const bool doc8 = FP8 && round * NSUB + j < n_doc;
        const int e = (hh * HD + ch0 + ln) * (doc8 ? 8 : 16) + (doc8 ? KBP : KB); // a channel's 8 keys follow each other
        const int step = doc8 ? 32 * 8 : 32 * 16;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            const gbl_char_t at = page_at(pg, rows_page_lane(round, j, s2));
#pragma unroll
            for (int mb = 0; mb < G::MBW; ++mb) vr[j % G::V_AHEAD][mb][s2] = ((gbl_word8_t)(at + e + mb * step))->w;
        }
    };
#pragma unroll
    for (int j = 0; j < G::V_AHEAD; ++j) load_v(cur, 0, j);
    Pages ahead = cur, nxt = cur;
    for (int r = 0;; ++r) {
        const int j0 = r * NSUB, n = n_sub - j0, l0 = (r & 1) * 2 * NSUB;
        if (r & 1) follow(ahead, nxt);
        lds_barrier();                                                            // the maxima are there
        lds_barrier();                                                            // P, the row sums and the factors are there
        constexpr int HALF = NSUB / 2;
        float alpha[HALF], sum[HALF];
        halfx8 pf[2][2];                                                          // two sub-tiles ahead
        auto load_p = [&](int j) {
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) pf[j % 2][s2] = *(const halfx8*)(smem + G::P_AT + j * 2048 + s2 * 1024 + lane * 16);
        };
        load_p(0);

#pragma unroll
        for (int j = 0; j < NSUB; ++j) {
            if (j == HALF && n <= j) break;                                       // the last round
            if (j % HALF == 0) {
#pragma unroll
                for (int i = 0; i < HALF; ++i) {
                    alpha[i] = s_alpha[(j + i) * 32 + ln];
                    sum[i] = s_sum[(j + i) * 64 + lane];
                }
            }
            if (j < n) {
                if (j + 1 < NSUB) load_p(j + 1);
                l_run = fmaf(l_run, alpha[j % HALF], sum[j % HALF]);
                if (__any(alpha[j % HALF] != 1.0f)) {
#pragma unroll
                    for (int mb = 0; mb < G::MBW; ++mb)
#pragma unroll
                        for (int e = 0; e < 16; ++e) oacc[mb][e] *= alpha[j % HALF];
                }
#pragma unroll
                for (int mb = 0; mb < G::MBW; ++mb) {
                    const uint4v a = vr[j % G::V_AHEAD][mb][0], b = vr[j % G::V_AHEAD][mb][1];
                    halfx8 v0 = __builtin_bit_cast(halfx8, a), v1 = __builtin_bit_cast(halfx8, b);
                    if (FP8 && j0 + j < n_doc) {
                        v0 = fp8x8_to_half(make_uint2(a[0], a[1]), fp8_expand_factor(lane_of(cur.sv, l0 + 2 * j)));
                        v1 = fp8x8_to_half(make_uint2(b[0], b[1]), fp8_expand_factor(lane_of(cur.sv, l0 + 2 * j + 1)));
                    }
                    oacc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(v0, pf[j % 2][0], oacc[mb], 0, 0, 0);
                    oacc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(v1, pf[j % 2][1], oacc[mb], 0, 0, 0);
                }
            }
            if (j < G::V_AHEAD) load_v(cur, r, j + G::V_AHEAD);
            else load_v(ahead, rows_asked(r + 1, rounds), j - G::V_AHEAD);
            asm volatile("" ::: "memory");                                        // the requests stay here, in front of the way out
        }
        if (r & 1) cur = ahead;
        if (rows_fetches_pages(r, rounds)) nxt = load_pages(r + 2);
        if (n <= NSUB) break;
    }
    const float inv = 1.0f / row_sum2(l_run);
    if (row < M) {
        const size_t orow = last_only ? (size_t)p : (size_t)(t0 + row_i);
        half_t* dst = o + (orow * n_kv * g + h * g + head) * HD + ch0 + 4 * hh;
#pragma unroll
        for (int mb = 0; mb < G::MBW; ++mb)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                halfx4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = from_float<half_t>(oacc[mb][r4 * 4 + e] * inv);
                *(halfx4*)(dst + mb * 32 + 8 * r4) = w;
            }
    }
}

template <int HD, bool FP8>
hipError_t launch_rows(const half_t* q, const char* kv_new, half_t* o, const MetaView& mv, const PoolView& pv, int layer, int n_q,
                       int last_only, int blocks, int max_keys, WeightWalks* warm, hipStream_t st) {
    if (!rows_holds(mv.n_seq, blocks)) return hipErrorInvalidValue;
    constexpr int kMaxDevices = 64;
    constexpr int lds = RowsGeo<HD>::LDS;
    static std::atomic<int> max_wgs_dev[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return hipErrorUnknown;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    int max_wgs = max_wgs_dev[dev].load(std::memory_order_acquire);
    if (max_wgs == 0) {
        hipError_t e = hipFuncSetAttribute((const void*)attn_rows_kernel<HD, FP8>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, attn_rows_kernel<HD, FP8>, kWaves * 64, lds) != hipSuccess || per_cu < 1)
            per_cu = 1;
        max_wgs = device_cu_count() * per_cu;
        max_wgs_dev[dev].store(max_wgs, std::memory_order_release);
    }
    // a row of workgroups per block: the blocks of a (sequence, kv head) lie on one XCD.  Then those that read weights ahead.
    const int items = (mv.n_seq * pv.n_kv + kXcds - 1) / kXcds * kXcds;
    WeightWalks walks;
    const int extra = warm ? pick_walks(warm, rows_warm_wgs(max_keys, FP8), max_wgs - items * blocks, &walks) : 0;
    const size_t layer_page0 = (size_t)layer * pv.num_pages * pv.n_kv;
    attn_rows_kernel<HD, FP8><<<dim3((unsigned)items, (unsigned)(blocks + (extra + items - 1) / items)), kWaves * 64, lds, st>>>(
        mv.cu, mv.prefix_len, mv.page_table, mv.new_cu, mv.pt_stride, pv.n_kv, make_divisor(pv.n_kv), n_q / pv.n_kv, make_divisor(n_q / pv.n_kv),
        (unsigned)mv.n_seq << 9 | (unsigned)blocks << 1 | (unsigned)last_only, q, kv_new, o,
        pv.data + layer_page0 * (2 * kPageTokens * HD * (FP8 ? 1 : 2)), FP8 ? pv.scales + layer_page0 * 2 : nullptr, extra, walks);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_rows(const void* q, const void* kv_new_pages, void* o, const MetaView& mv, const PoolView& pv, int layer, int n_q,
                            int blocks, int max_keys, hipStream_t st, bool last_only, WeightWalks* warm) {
    const half_t* qh = (const half_t*)q;
    const char* kvn = (const char*)kv_new_pages;
    half_t* oh = (half_t*)o;
    const bool fp8 = pv.kv_dtype == HR_FP8_E4M3;
    const int lo = last_only ? 1 : 0;
    if (pv.d == 64)
        return fp8 ? launch_rows<64, true>(qh, kvn, oh, mv, pv, layer, n_q, lo, blocks, max_keys, warm, st)
                   : launch_rows<64, false>(qh, kvn, oh, mv, pv, layer, n_q, lo, blocks, max_keys, warm, st);
    return fp8 ? launch_rows<128, true>(qh, kvn, oh, mv, pv, layer, n_q, lo, blocks, max_keys, warm, st)
               : launch_rows<128, false>(qh, kvn, oh, mv, pv, layer, n_q, lo, blocks, max_keys, warm, st);
}

}  // namespace hr
