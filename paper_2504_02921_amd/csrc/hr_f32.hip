// The fp32 pass: projections and attention of fp32 models on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32), plus
// the projections of 16-bit models whose shapes the half MFMA family does not cover (operands widened on load).
//
// fp32 models are small and their calls are short, so a launch is bound by latency (one pass over K is a few dependent
// loads), not by arithmetic.  Hence: operands go from global memory straight to registers in MFMA order (no LDS stage,
// no barrier in the k loop), the four wavefronts of a workgroup split K, a wavefront requests four 16-wide k-units at
// once, and the norm in front of a projection, RoPE and SwiGLU behind it are part of the projection's launch.
// Measured at 128 rows, hidden 256, ffn 688: the LDS-tiled VALU kernel these replace took 31-75 us per projection (2 x 12
// workgroups, 16 scalar loads per thread and k-step).
//
// Every output element is ((c0 + c2) + (c1 + c3)) of four chains, chain w over the 16-wide k-units w, w + 4, ..: the
// result does not depend on the tile shape or on the rows around it.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "hr_device_types.h"
#include "hr_kernels.h"
#include "hr_layout.h"

namespace hr {

typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(4))) _Float16 halfx4v;

namespace {

// Four consecutive operand values at k (a multiple of 4; every K is a multiple of 8).  Past the end of the row the address
// stays inside it; the caller clears one operand there.
template <typename T>
__device__ __forceinline__ floatx4 load4(const T* row, int k, int K) {
    const int kc = min(k, K - 4);
    if constexpr (sizeof(T) == 4) {
        return *(const floatx4*)(row + kc);
    } else {
        const halfx4v h = *(const halfx4v*)(row + kc);
        return floatx4{(float)h[0], (float)h[1], (float)h[2], (float)h[3]};
    }
}

// C = A W^T in 16 MI x 16 NI tiles, one workgroup of four wavefronts per tile.  MFMA orientation: W rows are the A
// operand, so a lane holds four consecutive columns of one output row and the partial tiles go to LDS as 16-byte words.
// The k order inside a 16-wide unit is permuted alike on both sides: lane group g holds k = 4 g + j for MFMA j, i.e. one
// 16-byte load per row and unit.
// UN: k-units of one pass of a wavefront's k loop.  The compiler puts a unit's loads in front of its MFMAs whatever their place here: one unit is
// in flight, and a unit is a trip to memory.
// NG: groups of four wavefronts beside each other, each with NI blocks of the tile's columns: a wavefront's MFMAs (16 x 16 x 4: 32 cycles
// each) are as long as its loads.
// What the loads need comes in front, as parameters of its own: 14 words are in scalar registers when a wavefront starts (kernarg preload).
template <typename T, F32Epilogue EPI, bool NORM, int MI, int NI, int UN, int NG>
__global__ void __launch_bounds__(256 * NG) gemm_f32_kernel(const void* A_, const void* W_, int M_, int N_, int K_, float eps_, const float* gain_,
                                                       F32GemmArgs rest) {
    F32GemmArgs a = rest;
    a.A = A_; a.W = W_; a.M = M_; a.N = N_; a.K = K_; a.eps = eps_; a.gain = gain_;
    constexpr int BM = 16 * MI, BN = 16 * NI * NG, LD = BN + 4, NT = 256 * NG;
    __shared__ __attribute__((aligned(16))) float part[2][BM * LD];
    __shared__ float row_ss[4][BM];
    const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & 3, grp = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int64_t m0 = (int64_t)blockIdx.x * BM;
    const int n0 = blockIdx.y * BN, col0 = 16 * NI * grp, K = a.K;
    const T *pa[MI], *pw[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) pa[i] = (const T*)a.A + min(m0 + 16 * i + r, a.M - 1) * K;
#pragma unroll
    for (int j = 0; j < NI; ++j) pw[j] = (const T*)a.W + (size_t)min(n0 + col0 + 16 * j + r, a.N - 1) * K;
    floatx4 acc[MI][NI];
    float ss[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        ss[i] = 0.f;
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const int units = (K + 15) / 16;
    for (int u0 = wave; u0 < units; u0 += 4 * UN) {
        floatx4 av[UN][MI], wv[UN][NI], gv[UN];
#pragma unroll
        for (int s = 0; s < UN; ++s) {
            const int k = (u0 + 4 * s) * 16 + 4 * kg;
#pragma unroll
            for (int i = 0; i < MI; ++i) av[s][i] = load4(pa[i], k, K);
#pragma unroll
            for (int j = 0; j < NI; ++j) wv[s][j] = load4(pw[j], k, K);
            if constexpr (NORM) gv[s] = ((const Loose<float, 4>*)(a.gain + min(k, K - 4)))->w;
        }
#pragma unroll
        for (int s = 0; s < UN; ++s) {
            const int k = (u0 + 4 * s) * 16 + 4 * kg;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = k < K ? av[s][i][e] : 0.f;
                    if constexpr (NORM) {
                        ss[i] = fmaf(x, x, ss[i]);
                        av[s][i][e] = x * gv[s][e];
                    } else {
                        av[s][i][e] = x;
                    }
                }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[s][j][e], av[s][i][e], acc[i][j], 0, 0, 0);
        }
    }
    // the four chains of an element: waves 2, 3 -> LDS, waves 0, 1 add theirs, everybody reads the two sums
    if constexpr (NORM) {
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            ss[i] += __shfl_xor(ss[i], 16, 64);
            ss[i] += __shfl_xor(ss[i], 32, 64);
            if (kg == 0 && grp == 0) row_ss[wave][16 * i + r] = ss[i];
        }
    }
    float* mine = part[wave & 1];
    auto at = [&](int i, int j) { return (floatx4*)(mine + (16 * i + r) * LD + col0 + 16 * j + 4 * kg); };
    if (wave >= 2) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) *at(i, j) = acc[i][j];
    }
    __syncthreads();
    if (wave < 2) {                                // a lane reads back and replaces its own element positions
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) *at(i, j) = acc[i][j] + *at(i, j);
    }
    __syncthreads();
    auto row_scale = [&](int m) {
        if constexpr (!NORM) return 1.0f;
        return 1.0f / sqrtf(((row_ss[0][m] + row_ss[1][m]) + (row_ss[2][m] + row_ss[3][m])) / (float)K + a.eps);
    };
    auto value = [&](int m, int n) { return part[0][m * LD + n] + part[1][m * LD + n]; };
    if constexpr (EPI == F32_STORE || EPI == F32_ADD) {
#pragma unroll
        for (int e0 = 0; e0 < BM * BN; e0 += NT) {
            const int e = e0 + threadIdx.x, m = e / BN, n = e % BN;
            const int64_t row = m0 + m;
            if (row >= a.M || n0 + n >= a.N) continue;
            float* c = a.C + row * a.N + n0 + n;
            const float v = value(m, n) * row_scale(m);
            if constexpr (EPI == F32_ADD) *c = a.add_rows ? a.add[(size_t)a.add_rows[row] * a.N + n0 + n] + v : *c + v;
            else *c = v;
        }
    } else if constexpr (EPI == F32_ROPE) {        // BN is a multiple of the head size: whole heads per tile
        const int d = a.d, half = d / 2, rot = a.n_q + a.n_kv;
#pragma unroll
        for (int e0 = 0; e0 < BM * BN / 2; e0 += NT) {
            const int e = e0 + threadIdx.x, m = e / (BN / 2), p = e % (BN / 2);
            const int lh = p / half, j = p - lh * half;
            const int64_t row = m0 + m;
            const int hd = n0 / d + lh;
            if (row >= a.M || hd * d >= a.N) continue;
            const float rs = row_scale(m);
            float x1 = value(m, lh * d + j) * rs, x2 = value(m, lh * d + j + half) * rs;
            if (hd < rot) {
                const float2 cs = a.rope[row * half + j];
                const float o1 = rope_lo(x1, x2, cs.x, cs.y), o2 = rope_hi(x1, x2, cs.x, cs.y);
                x1 = o1;
                x2 = o2;
            }
            float* dst = hd < a.n_q ? a.q + (row * a.n_q + hd) * d
                                    : (hd < rot ? a.k + (row * a.n_kv + (hd - a.n_q)) * d : a.v + (row * a.n_kv + (hd - rot)) * d);
            dst[j] = x1;
            dst[j + half] = x2;
        }
    } else {                                       // F32_SWIGLU: BN is a multiple of a gate block and its up block
        const int F = a.N / 2, ib = a.ib;
#pragma unroll
        for (int e0 = 0; e0 < BM * BN / 2; e0 += NT) {
            const int e = e0 + threadIdx.x, m = e / (BN / 2), fl = e % (BN / 2);
            const int64_t row = m0 + m;
            const int f = n0 / 2 + fl, base = (fl / ib) * 2 * ib + fl % ib;
            if (row >= a.M || f >= F) continue;
            const float rs = row_scale(m);
            const float g = value(m, base) * rs, u = value(m, base + ib) * rs;
            a.C[row * F + f] = g / (1.0f + expf(-g)) * u;
        }
    }
}

template <typename T, F32Epilogue EPI, bool NORM, int MI, int NI, int UN, int NG = 1>
hipError_t launch_f32_tile(const F32GemmArgs& a, hipStream_t st) {
    const dim3 grid((unsigned)((a.M + 16 * MI - 1) / (16 * MI)), (unsigned)((a.N + 16 * NI * NG - 1) / (16 * NI * NG)));
    gemm_f32_kernel<T, EPI, NORM, MI, NI, UN, NG><<<grid, 256 * NG, 0, st>>>(a.A, a.W, (int)a.M, a.N, a.K, a.eps, a.gain, a);
    return hipGetLastError();
}

// Tile shape: 64 x 64 (an operand value is used 64 times) once that gives most CUs a workgroup, else 16 rows, so that
// short launches spread over the chip: 16 columns, or 64 where the epilogue needs whole heads / gate-up block pairs.
template <typename T, F32Epilogue EPI, bool NORM>
hipError_t launch_f32_shape(const F32GemmArgs& a, hipStream_t st) {
    const int64_t big = ((a.M + 63) / 64) * ((a.N + 63) / 64);
    if (big >= 192) return launch_f32_tile<T, EPI, NORM, 4, 4, 2>(a, st);
    if constexpr (EPI == F32_STORE || EPI == F32_ADD) {
        return launch_f32_tile<T, EPI, NORM, 1, 1, 4>(a, st);
    } else {
        // two groups of wavefronts where a CU has one workgroup at most: 128 tokens, hidden 256, ffn 688 (96 and 176 workgroups) 7.1 -> 6.5 us a
        // launch, the call 71.4 -> 69.1; 480 tokens (360 and 660) 104 -> 106 us a call
        if (((a.M + 15) / 16) * ((a.N + 63) / 64) <= device_cu_count()) return launch_f32_tile<T, EPI, NORM, 1, 2, 4, 2>(a, st);
        return launch_f32_tile<T, EPI, NORM, 1, 4, 4>(a, st);
    }
}

// ---- prefix + causal attention of fp32 models.  One workgroup per (sequence, kv head, 16 query rows); its wavefronts take
// the 16-key tiles (one pool page, or 16 new tokens) in turn, each with an online softmax of its own, and merge through
// LDS at the end.  Scores are computed transposed (S^T = K Q^T): a lane owns one query row and four keys, which is
// the B-operand order of O^T += V^T P^T, so the probabilities never leave the registers.  K, Q and V are read in 16-byte
// words straight from the pages.  8 sequences x 128 + 16 keys, 4 heads: one lane per key with scalar loads took 35 us.
// Rows are token-major with g heads per token; last_only: the g rows of the last token, written compactly.
template <int D, int NW>
__global__ void __launch_bounds__(NW * 64) attn_f32_kernel(const int32_t* __restrict__ m_cu, const int32_t* __restrict__ m_prefix,
                                                           const int32_t* __restrict__ m_pt, int pt_stride, int n_q, int n_kv, int last_only,
                                                           const float* __restrict__ q, const float* __restrict__ layer_data,
                                                           const float* __restrict__ k_new, const float* __restrict__ v_new,
                                                           float* __restrict__ o, int block0) {
    constexpr int CB = D / 16, LD = D + 4;
    __shared__ __attribute__((aligned(16))) float so[NW][16 * LD];
    __shared__ float sml[2][NW][16];
    const int lane = threadIdx.x & 63, r = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int p = blockIdx.x, h = blockIdx.y, g = n_q / n_kv;
    const int t0 = m_cu[p], q_len = m_cu[p + 1] - t0, Dl = m_prefix[p];
    const int row_first = last_only ? (q_len - 1) * g : 0, rows = last_only ? g : q_len * g;
    const int row0 = (block0 + (int)blockIdx.z) * 16;
    if (row0 >= rows) return;
    const int row = row_first + min(row0 + r, rows - 1);       // this lane's query row
    const int tok = row / g;
    const float* qr = q + ((size_t)(t0 + tok) * n_q + h * g + (row - tok * g)) * D;
    floatx4 qv[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) qv[c] = *(const floatx4*)(qr + c * 16 + 4 * kg);
    const float scale = 1.0f / sqrtf((float)D);
    const int32_t* pt = m_pt + (size_t)p * pt_stride;
    const int n_pages = (Dl + kPageTokens - 1) / kPageTokens;
    const int tok_last = (row_first + min(row0 + 15, rows - 1)) / g;
    const int n_tiles = n_pages + tok_last / 16 + 1;
    floatx4 acc[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
    float mx = -INFINITY, sum = 0.f;
    for (int tile = wave; tile < n_tiles; tile += NW) {
        floatx4 kv[CB], vv[CB];
        int lim;                                               // key j of the tile is visible where j <= lim
        if (tile < n_pages) {
            const float* kb = layer_data + ((size_t)pt[tile] * n_kv + h) * (2 * kPageTokens * D);
            const float* vb = kb + kPageTokens * D;
            lim = Dl - 1 - tile * 16;
#pragma unroll
            for (int c = 0; c < CB; ++c) kv[c] = *(const floatx4*)(kb + k_elem(r, c * 16 + 4 * kg, D, 4));
#pragma unroll
            for (int c = 0; c < CB; ++c) vv[c] = *(const floatx4*)(vb + v_elem(4 * kg, c * 16 + r, D));     // keys 4 kg .. + 3
            if (lim < kPageTokens - 1) {                       // the document ends inside this page: what lies behind may be infinite
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (4 * kg + e > lim) {
#pragma unroll
                        for (int c = 0; c < CB; ++c) vv[c][e] = 0.f;
                    }
            }
        } else {
            const int j0 = (tile - n_pages) * 16;
            lim = tok - j0;
            const float* kb = k_new + ((size_t)(t0 + min(j0 + r, q_len - 1)) * n_kv + h) * D;
#pragma unroll
            for (int c = 0; c < CB; ++c) kv[c] = *(const floatx4*)(kb + c * 16 + 4 * kg);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float* vb = v_new + ((size_t)(t0 + min(j0 + 4 * kg + e, q_len - 1)) * n_kv + h) * D;
#pragma unroll
                for (int c = 0; c < CB; ++c) vv[c][e] = vb[c * 16 + r];
            }
        }
        floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[c][e], qv[c][e], s, 0, 0, 0);
        float tm = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[e] = 4 * kg + e <= lim ? s[e] * scale : -INFINITY;
            tm = fmaxf(tm, s[e]);
        }
        tm = fmaxf(tm, __shfl_xor(tm, 16, 64));
        tm = fmaxf(tm, __shfl_xor(tm, 32, 64));
        const float nm = fmaxf(mx, tm), base = nm == -INFINITY ? 0.f : nm;
        const float f = expf(mx - base);                       // 0 before the first visible key
        float ts = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[e] = expf(s[e] - base);
            ts += s[e];
        }
        sum = sum * f + ts;
        mx = nm;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            acc[c] *= f;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[c][e], s[e], acc[c], 0, 0, 0);
        }
    }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    if (kg == 0) {
        sml[0][wave][r] = mx;
        sml[1][wave][r] = sum;
    }
#pragma unroll
    for (int c = 0; c < CB; ++c) *(floatx4*)(so[wave] + r * LD + c * 16 + 4 * kg) = acc[c];
    __syncthreads();
    for (int e = threadIdx.x; e < 16 * D; e += NW * 64) {
        const int er = e / D, c = e % D;
        if (row0 + er >= rows) continue;
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) m = fmaxf(m, sml[0][w][er]);
        float num = 0.f, den = 0.f;                            // a row always sees its own key: m is finite
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = expf(sml[0][w][er] - m);
            num = fmaf(f, so[w][er * LD + c], num);
            den = fmaf(f, sml[1][w][er], den);
        }
        const int rr = row_first + row0 + er, tk = rr / g;
        const size_t out_tok = last_only ? (size_t)p : (size_t)(t0 + tk);
        o[(out_tok * n_q + h * g + (rr - tk * g)) * D + c] = num / den;
    }
}

}  // namespace

hipError_t launch_gemm_f32(F32Epilogue epi, int dtype, const F32GemmArgs& a, hipStream_t st) {
    if (a.M == 0) return hipSuccess;
    if (a.K % 8 != 0) return hipErrorInvalidValue;
    if (dtype != HR_F32) {                         // half operands, fp32 result
        if (epi == F32_STORE && !a.gain) return launch_f32_shape<half_t, F32_STORE, false>(a, st);
        if (epi == F32_ADD && !a.gain) return launch_f32_shape<half_t, F32_ADD, false>(a, st);
        return hipErrorInvalidValue;
    }
    switch (epi) {
        case F32_STORE: if (!a.gain) return launch_f32_shape<float, F32_STORE, false>(a, st); break;
        case F32_ADD: if (!a.gain) return launch_f32_shape<float, F32_ADD, false>(a, st); break;
        case F32_ROPE: if (a.gain && 64 % a.d == 0) return launch_f32_shape<float, F32_ROPE, true>(a, st); break;
        case F32_SWIGLU: if (a.gain && (a.ib == 32 || a.ib == 1)) return launch_f32_shape<float, F32_SWIGLU, true>(a, st); break;
    }
    return hipErrorInvalidValue;
}

bool f32_fused_supported(const hr_model_cfg& c) {
    return c.dtype == HR_F32 && (c.head_dim == 16 || c.head_dim == 32 || c.head_dim == 64);
}

hipError_t launch_attn_f32(const float* q, const float* k_new, const float* v_new, float* o, const MetaView& mv, const PoolView& pv,
                           int layer, int n_q, int max_q_len, bool last_only, hipStream_t st) {
    if (mv.T == 0) return hipSuccess;
    const int g = n_q / pv.n_kv;
    const int64_t rows = last_only ? g : (int64_t)g * max_q_len;
    // one launch as a rule: a grid holds 65535 row blocks in its third dimension
    const int64_t blocks = (rows + 15) / 16;
    const float* layer_data = (const float*)pv.data + (size_t)layer * pv.num_pages * pv.n_kv * (2 * kPageTokens * pv.d);
#define HR_ATTN_F32(D)                                                                                                                  \
    attn_f32_kernel<D, 8><<<grid, 512, 0, st>>>(mv.cu, mv.prefix_len, mv.page_table, mv.pt_stride, n_q, pv.n_kv, last_only, q, layer_data, \
                                                k_new, v_new, o, (int)b0)
    for (int64_t b0 = 0; b0 < blocks; b0 += 65535) {
        const dim3 grid((unsigned)mv.n_seq, (unsigned)pv.n_kv, (unsigned)std::min<int64_t>(blocks - b0, 65535));
        switch (pv.d) {
            case 16: HR_ATTN_F32(16); break;
            case 32: HR_ATTN_F32(32); break;
            case 64: HR_ATTN_F32(64); break;
            default: return hipErrorInvalidValue;
        }
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
#undef HR_ATTN_F32
    return hipSuccess;
}

}  // namespace hr
