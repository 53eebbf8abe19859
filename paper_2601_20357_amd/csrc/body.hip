// Draft-model body in front of the LM head (Sec. 5.1 "Ensemble learning via Batched Inference", Sec. 4.1 "Target and
// Draft Models"): one decode step of a LLaMA-style decoder for the n*B rows of the batch of drafting methods, each
// with its own key / value cache.  Up to 16 rows the step is one launch where its sizes allow (body_gang.hip); here are the
// others.  At 64 rows every projection streams a few megabytes of weights and is bound by
// launch and latency, not bandwidth, so a layer is five launches and nothing in between: every projection normalises
// (or merges the attention's partial results) while its weights are on their way and finishes what its result feeds --
// rotation and cache append, residual addition, SwiGLU -- before it stores.  Storage points: bf16 for weights, caches
// and everything that feeds a projection; fp32 for the residual stream, the rotated queries and the attention's
// partial sums.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <mutex>
#include <utility>

#include "body_utils.h"
#include "device_utils.h"
#include "internal.h"

namespace tabed {

__device__ __forceinline__ float block_sum_f32(float v, float* lds4) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) lds4[threadIdx.x >> 6] = v;
    __syncthreads();
    const float r = (lds4[0] + lds4[1]) + (lds4[2] + lds4[3]);
    __syncthreads();
    return r;
}

// ---------------------------------------------------------------- embedding
// The second half of the workgroup's work: cos and sin of the row's position times every rotation frequency, which all
// layers share, in fp64 (a position times a tiny frequency loses digits in fp32).
__global__ __launch_bounds__(kBlock) void k_body_embed(int d, int V, const int32_t* __restrict__ token_src, int token_stride,
                                                       int rows_per_token, const uint16_t* __restrict__ embed,
                                                       float* __restrict__ x, const int32_t* __restrict__ ctx_len, int max_ctx,
                                                       int hd, double log2_theta, double2* __restrict__ trig /* [rows][hd/2] */,
                                                       uint64_t* __restrict__ gang_key, float* __restrict__ ones /* [rows] or null */) {
    const int r = blockIdx.x;
    if (ones != nullptr && threadIdx.x == 0) ones[r] = 1.f;     // each step: a step of fewer rows may have had the workspace in between
    if (r == 0 && threadIdx.x == 0) *gang_key = 0;      // a one-launch step on the same workspace finds its buffers used otherwise
    const int pos = min(max(ctx_len[r], 0), max_ctx - 1);
    int tok = token_src[(size_t)(r / rows_per_token) * token_stride];
    tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
    const uint16_t* e = embed + (size_t)tok * d;
    for (int i = threadIdx.x; i < d / 8; i += kBlock) {
        const u32x4b w = *reinterpret_cast<const u32x4b*>(e + 8 * i);
        float4* xp = reinterpret_cast<float4*>(x + (size_t)r * d + 8 * i);
        auto lo = [&](int q) { return __builtin_bit_cast(float, w[q] << 16); };
        auto hi = [&](int q) { return __builtin_bit_cast(float, w[q] & 0xffff0000u); };
        xp[0] = make_float4(lo(0), hi(0), lo(1), hi(1));
        xp[1] = make_float4(lo(2), hi(2), lo(3), hi(3));
    }
    const int i = kBlock - 1 - threadIdx.x;                                // hd / 2 <= 64 angles: the last wave's lanes
    if (i < hd / 2) {
        double sn, cs;
        sincos((double)pos * exp2(-2.0 * (double)i / (double)hd * log2_theta), &sn, &cs);
        trig[(size_t)r * (hd / 2) + i] = make_double2(cs, sn);
    }
}

// ---------------------------------------------------------------- RMSNorm of the residual stream (+ position advance at the end of a step)
__global__ __launch_bounds__(kBlock) void k_body_norm(int d, float eps, const float* __restrict__ x, const float* __restrict__ g,
                                                      uint16_t* __restrict__ out, int32_t* __restrict__ ctx_len_advance) {
    __shared__ float s_red[kWavesPerBlock];
    const int r = blockIdx.x;
    const float4* xr = reinterpret_cast<const float4*>(x + (size_t)r * d);
    float ss = 0.f;
    for (int i = threadIdx.x; i < d / 4; i += kBlock) {
        const float4 v = xr[i];
        ss += (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
    }
    const float inv = 1.f / sqrtf(block_sum_f32(ss, s_red) / (float)d + eps);
    for (int i = threadIdx.x; i < d / 4; i += kBlock) {
        const float4 v = xr[i];
        const float4 gg = *reinterpret_cast<const float4*>(g + 4 * i);
        *reinterpret_cast<uint2*>(out + (size_t)r * d + 4 * i) = pack_bf16x4(v.x * inv * gg.x, v.y * inv * gg.y, v.z * inv * gg.z, v.w * inv * gg.w);
    }
    if (ctx_len_advance != nullptr && threadIdx.x == 0) ctx_len_advance[r] += 1;
}

// ---------------------------------------------------------------- projections
// One workgroup = 16 * MB rows and one 16-column tile of the result (two tiles that belong together for the rotation and
// for SwiGLU), over the whole contraction: its waves take k-blocks of 64 in turn and meet through LDS, where the results are
// added in wave order.  A wave reads W as whole 128-byte lines, 8 lanes a row, and turns every k-block through a private LDS
// patch into the operand layout of v_mfma_f32_16x16x32_bf16 (read straight into that layout, 16 consecutive lanes hold 16
// different rows and a load instruction looks up 64 lines instead of 8).  Everything a wave needs is requested before
// anything is used (G = k-blocks a wave requests together), what is needed first first.
//   IN  kInNorm:    X = bf16(x * inv_rms * g): a wave reads whole rows of the residual stream (CI pieces of 256 columns),
//                   so that it has their sums of squares, and leaves the rows in LDS
//       kInBf16:    X as it is, through the patch like W
//       kInMerge:   X = the attention's partial results of `splits` key ranges, merged into LDS
//   EPI kEpiRope:   q/k/v columns: rotation in fp64, queries to `q`, the new key and value to the caches
//       kEpiSilu:   gate and up columns of the same 16 units: silu(gate) * up
//       kEpiAdd:    residual addition in place
// At 64 rows of d = 768, d_ff = 3072 a launch moves 1 to 9 MB: latency, the rate at which a compute unit takes in W and X
// (64 bytes a cycle: every workgroup reads its rows of X whole) and the instructions fetched once bound it.  Measured
// there (kernel trace, average): q/k/v 7.2, o 4.6, gate/up 10.0, down 5.9 us (down 8.0 with loads straight into operand
// layout); with the contraction split over workgroups, partial sums in memory and rotation, residual + norm and SwiGLU kernels
// of their own a layer took 62 us instead of 48.
enum { kInNorm = 0, kInBf16 = 1, kInMerge = 2 };
enum { kEpiRope = 0, kEpiSilu = 1, kEpiAdd = 2 };

struct ProjArgs {
    int M, N, K;                 // rows, columns of the result (kEpiSilu: units), contraction
    const uint16_t* W;
    const uint16_t* X;           // kInBf16: [M,K]
    float* x;                    // residual stream [M,d]: read by kInNorm, updated by kEpiAdd
    const float* g;              // kInNorm
    float eps;
    const float* po;             // kInMerge: [splits][M,K] sums of p * v, not normalised
    const float* pml;            // kInMerge: [M][heads][splits][2] maximum (base 2) and sum of p
    int splits, hd;
    float* q;                    // kEpiRope: [M,d]
    uint16_t* kc;
    uint16_t* vc;
    const int32_t* ctx_len;
    int max_ctx;
    const double2* trig;         // kEpiRope: [M][hd/2] cos, sin of the rows' positions
    uint16_t* act;               // kEpiSilu: [M,N]
};

constexpr int kBodyPatch = 16 * 144;                  // bytes: 16 rows of one k-block, padded

__host__ __device__ constexpr int staged_row(int K) { return (K + 63) / 64 * 64 + 8; }   // bf16 of one staged row of X, padded

// kInMerge: the rows' attention output, merged over SP key ranges, U pieces of four columns per thread in flight.
template <int SP, int U>
__device__ __forceinline__ void merge_splits(const ProjArgs& a, int m0, int threads, uint16_t* s_x) {
    const int xrow = staged_row(a.K), per_row = (a.K + 63) / 64 * 16, heads = a.K / a.hd, total = min(16, a.M - m0) * per_row;
    for (int u0 = threadIdx.x; u0 < total; u0 += threads * U) {
        float4 o[U][SP];
        float2 ml[U][SP];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = min(u0 + u * threads, total - 1), m = m0 + idx / per_row, k = min((idx % per_row) * 4, a.K - 4);
#pragma unroll
            for (int s = 0; s < SP; ++s) {
                ml[u][s] = *reinterpret_cast<const float2*>(a.pml + (((size_t)m * heads + k / a.hd) * SP + s) * 2);
                o[u][s] = *reinterpret_cast<const float4*>(a.po + ((size_t)s * a.M + m) * a.K + k);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = u0 + u * threads;
            float M = ml[u][0].x;
#pragma unroll
            for (int s = 1; s < SP; ++s) M = fmaxf(M, ml[u][s].x);
            float L = 0.f;
            float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int s = 0; s < SP; ++s) {
                const float w = __builtin_amdgcn_exp2f(ml[u][s].x - M);
                L += ml[u][s].y * w;
                t.x += o[u][s].x * w; t.y += o[u][s].y * w; t.z += o[u][s].z * w; t.w += o[u][s].w * w;
            }
            if (idx < total) {
                const int row = idx / per_row, k = (idx % per_row) * 4;
                const float inv = 1.f / L;
                *reinterpret_cast<uint2*>(s_x + row * xrow + k) = k < a.K ? pack_bf16x4(t.x * inv, t.y * inv, t.z * inv, t.w * inv) : make_uint2(0u, 0u);
            }
        }
    }
}

template <int NW, int MB, int G, int CI, int IN, int EPI>
__global__ __launch_bounds__(NW * 64) void k_body_proj(ProjArgs a) {
    constexpr int NB = (EPI == kEpiAdd) ? 1 : 2;
    constexpr int kThreads = NW * 64;
    constexpr int kElems = (MB * 256 + kThreads - 1) / kThreads;          // result positions (or pairs) per thread
    constexpr int RW = MB * 16 / NW;                                      // kInNorm: rows a wave stages
    static_assert(IN != kInMerge || MB == 1, "the merge stages 16 rows");
    // staged rows of X, the waves' patches, then (after a barrier) their results [NW][NB][MB][16][20]
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];
    uint16_t* const s_x = reinterpret_cast<uint16_t*>(s_dyn);
    float* const s_acc = reinterpret_cast<float*>(s_dyn);
    const int tile = blockIdx.x, m0 = blockIdx.y * (MB * 16), tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, c = lane >> 4, lrow = lane >> 3, lchunk = lane & 7, K = a.K, KB = (K + 63) / 64, xrow = staged_row(K);
    constexpr int kPatches = NB + ((IN == kInBf16) ? MB : 0);
    unsigned char* const patch = s_dyn + ((IN == kInBf16) ? 0 : MB * 16 * xrow * 2) + wave * (kPatches * kBodyPatch);

    // which columns: [part][d] for q/k/v; the second tile is the rotation's other half, the up column, or the next 16
    int col0 = tile * 16, col1 = 0, lim0 = a.N, part = 0, j0 = 0;
    if (EPI == kEpiRope) {
        const int d = a.N / 3, per_part = (d + 31) / 32;
        part = tile / per_part;
        const int t = tile % per_part;
        if (a.hd >= 32) {
            const int per_head = a.hd / 32, head = t / per_head;
            j0 = (t % per_head) * 16;
            col0 = part * d + head * a.hd + j0;
            col1 = col0 + a.hd / 2;
        } else {
            j0 = t * 32;                                                  // first of 32 adjacent columns: whole heads
            col0 = part * d + j0;
            col1 = col0 + 16;
        }
        lim0 = part * d + d;
    } else if (EPI == kEpiSilu) {
        col1 = a.N + col0;
    }
    // uniform bases and 32-bit lane offsets (in bytes): a load is one instruction with no 64-bit address arithmetic
    const char* wb[NB];
    uint32_t wo[NB][2], xo[MB][2];                                        // [rows 8 i + lane / 8 of the tile]
    wb[0] = reinterpret_cast<const char*>(a.W) + (size_t)col0 * K * 2;
    int last0 = lim0 - 1 - col0, last1 = 0;                               // last row of W that a tile may read
    if (NB == 2) {                                                        // (hd < 32: the second 16 columns may start past the part)
        const int lim1 = (EPI == kEpiSilu) ? 2 * a.N : lim0, first = min(col1, lim1 - 1);
        wb[NB - 1] = reinterpret_cast<const char*>(a.W) + (size_t)first * K * 2;
        last1 = lim1 - 1 - first;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        wo[0][i] = (uint32_t)min(8 * i + lrow, last0) * (uint32_t)K * 2u;
        if (NB == 2) wo[NB - 1][i] = (uint32_t)min(8 * i + lrow, last1) * (uint32_t)K * 2u;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) xo[mb][i] = (uint32_t)min(mb * 16 + 8 * i + lrow, a.M - 1 - m0) * (uint32_t)K * 2u;
    }

    // ---- requests, in the order of use
    int pos[kElems];
    if (EPI == kEpiRope) {
#pragma unroll
        for (int e = 0; e < kElems; ++e) pos[e] = a.ctx_len[min(m0 + ((tid + e * kThreads) >> 4), a.M - 1)];
    }
    f32x4b xr[(IN == kInNorm) ? RW : 1][(IN == kInNorm) ? CI : 1], gr[(IN == kInNorm) ? CI : 1];
    if (IN == kInNorm) {
        const char* xbase = reinterpret_cast<const char*>(a.x) + (size_t)m0 * K * 4;
#pragma unroll
        for (int i = 0; i < CI; ++i) {
            const uint32_t k = (uint32_t)min((i * 64 + lane) * 4, K - 4) * 4u;
#pragma unroll
            for (int r = 0; r < RW; ++r)
                if (m0 + wave + r * NW < a.M)                             // uniform: rows that are not there are not read
                    xr[r][i] = *reinterpret_cast<const f32x4b*>(xbase + (size_t)((wave + r * NW) * K) * 4 + k);
        }
#pragma unroll
        for (int i = 0; i < CI; ++i)
            gr[i] = *reinterpret_cast<const f32x4b*>(reinterpret_cast<const char*>(a.g) + (uint32_t)min((i * 64 + lane) * 4, K - 4) * 4u);
        __builtin_amdgcn_sched_barrier(0);
    }
    u32x4b wv[G][NB][2], xb[(IN == kInBf16) ? G : 1][MB][2];
    auto request = [&](int b0) {
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int kb = min(b0 + q * NW, KB - 1);                      // past the last block: re-read, not used
            const uint32_t k = min((uint32_t)(kb * 128 + lchunk * 16), (uint32_t)K * 2u - 16u);   // past the last column: zeroed below
            const char* const xbase = reinterpret_cast<const char*>(a.X) + (size_t)m0 * K * 2;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) wv[q][nb][i] = *reinterpret_cast<const u32x4b*>(wb[nb] + (wo[nb][i] + k));
                if (IN == kInBf16) {
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) xb[q][mb][i] = *reinterpret_cast<const u32x4b*>(xbase + (xo[mb][i] + k));
                }
            }
        }
    };
    request(wave);
    float xold[kElems];                                                   // kEpiAdd: the residual stream's entries of this thread
    if (EPI == kEpiAdd) {
#pragma unroll
        for (int e = 0; e < kElems; ++e) {
            const int idx = tid + e * kThreads;
            xold[e] = a.x[(size_t)min(m0 + (idx >> 4), a.M - 1) * a.N + min(col0 + (idx & 15), a.N - 1)];
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- while W is on its way: the staged rows
    if (IN == kInNorm) {
        float mine = 0.f;                                                 // lane r: row r's sum of squares, then 1 / rms
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            float ss = 0.f;
#pragma unroll
            for (int i = 0; i < CI; ++i) {
                const f32x4b v = xr[r][i];
                const float t = (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
                ss += ((i * 64 + lane) * 4 < K) ? t : 0.f;
            }
            ss = wave_sum(ss);
            mine = (lane == r) ? ss : mine;
        }
        mine = 1.f / sqrtf(mine / (float)K + a.eps);
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const float inv = lane_f32(mine, r);
#pragma unroll
            for (int i = 0; i < CI; ++i) {
                const int k = (i * 64 + lane) * 4;
                const f32x4b v = xr[r][i];
                if (k < KB * 64)
                    *reinterpret_cast<uint2*>(s_x + (wave + r * NW) * xrow + k) =
                        k < K ? pack_bf16x4(v[0] * inv * gr[i][0], v[1] * inv * gr[i][1], v[2] * inv * gr[i][2], v[3] * inv * gr[i][3])
                              : make_uint2(0u, 0u);
            }
        }
    }
    if (IN == kInMerge) {
        if (a.splits == 2) merge_splits<2, 6>(a, m0, kThreads, s_x);
        else if (a.splits == 4) merge_splits<4, 3>(a, m0, kThreads, s_x);
        else merge_splits<8, 2>(a, m0, kThreads, s_x);
    }
    double2 cs[kElems];
    int ia[kElems], ib[kElems];                                           // columns (0..31 of the two tiles) of a pair
    if (EPI == kEpiRope) {
        const int half = a.hd / 2;
#pragma unroll
        for (int e = 0; e < kElems; ++e) {
            const int n = (tid + e * kThreads) & 15;
            pos[e] = pos[e] < 0 ? 0 : (pos[e] >= a.max_ctx ? a.max_ctx - 1 : pos[e]);   // never write outside the row's cache
            ia[e] = (a.hd >= 32) ? n : (n / half) * a.hd + n % half;
            ib[e] = (a.hd >= 32) ? n + 16 : ia[e] + half;
            cs[e] = a.trig[(size_t)min(m0 + ((tid + e * kThreads) >> 4), a.M - 1) * half + ((a.hd >= 32) ? j0 + n : n % half)];
        }
    }
    if (IN != kInBf16) lds_barrier();

    f32x4b acc[NB][MB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = f32x4b{0.f, 0.f, 0.f, 0.f};
    for (int b0 = wave; b0 < KB; b0 += NW * G) {
        if (b0 != wave) request(b0);
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int kb = b0 + q * NW;
            if (kb < KB) {                                                // LDS operations of one wave execute in order: no barrier
                const bool out = kb * 64 + lchunk * 8 >= K;               // K is a multiple of 8: a piece is in or out
                const u32x4b zero = {0u, 0u, 0u, 0u};
                unsigned char* const to = patch + lrow * 144 + lchunk * 16;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) *reinterpret_cast<u32x4b*>(to + nb * kBodyPatch + i * 8 * 144) = out ? zero : wv[q][nb][i];
                    if (IN == kInBf16) {
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
                            *reinterpret_cast<u32x4b*>(to + (NB + mb) * kBodyPatch + i * 8 * 144) = out ? zero : xb[q][mb][i];
                    }
                }
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const unsigned char* const from = patch + r16 * 144 + p * 64 + c * 16;
                    bf16x8 w[NB];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) w[nb] = *reinterpret_cast<const bf16x8*>(from + nb * kBodyPatch);
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) {
                        const bf16x8 xv = (IN == kInBf16) ? *reinterpret_cast<const bf16x8*>(from + (NB + mb) * kBodyPatch)
                                        : *reinterpret_cast<const bf16x8*>(s_x + (IN == kInMerge ? min(r16, a.M - 1 - m0) : mb * 16 + r16) * xrow +
                                                                           kb * 64 + p * 32 + c * 8);
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            acc[nb][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[nb], xv, acc[nb][mb], 0, 0, 0);
                    }
                }
            }
        }
    }
    __syncthreads();                                                      // every wave is done with the staged rows and its patch
    // accumulator: lane holds row r16 of the block, columns 4 c .. 4 c + 3 of the tile
    auto slot_of = [&](int w, int nb, int mb, int row, int col) { return (((w * NB + nb) * MB + mb) * 16 + row) * 20 + col; };
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) *reinterpret_cast<f32x4b*>(s_acc + slot_of(wave, nb, mb, r16, 4 * c)) = acc[nb][mb];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kElems; ++e) {
        const int idx = tid + e * kThreads;
        if (idx >= MB * 256) break;
        const int mb = idx >> 8, ml = (idx >> 4) & 15, n = idx & 15, m = m0 + mb * 16 + ml;
        auto total = [&](int col) {
            float t = s_acc[slot_of(0, col >> 4, mb, ml, col & 15)];
#pragma unroll
            for (int w = 1; w < NW; ++w) t += s_acc[slot_of(w, col >> 4, mb, ml, col & 15)];
            return t;
        };
        if (m >= a.M) continue;
        if (EPI == kEpiAdd) {
            const int col = col0 + n;
            if (col < a.N) a.x[(size_t)m * a.N + col] = xold[e] + total(n);
        } else if (EPI == kEpiSilu) {
            const int col = col0 + n;
            if (col < a.N) {
                const float gte = total(n), up = total(16 + n);
                a.act[(size_t)m * a.N + col] = f32_to_bf16_bits(gte / (1.f + __expf(-gte)) * up);
            }
        } else {
            const int d = a.N / 3;
            const int ca = (a.hd >= 32) ? col0 - part * d + n : j0 + ia[e], cb = (a.hd >= 32) ? ca + a.hd / 2 : j0 + ib[e];
            if (cb < d) {
                const float v0 = total(ia[e]), v1 = total(ib[e]);
                const size_t slot = ((size_t)m * a.max_ctx + pos[e]) * d;
                if (part == 2) {
                    a.vc[slot + ca] = f32_to_bf16_bits(v0);
                    a.vc[slot + cb] = f32_to_bf16_bits(v1);
                } else {
                    const float y0 = (float)((double)v0 * cs[e].x - (double)v1 * cs[e].y), y1 = (float)((double)v1 * cs[e].x + (double)v0 * cs[e].y);
                    if (part == 0) {
                        a.q[(size_t)m * d + ca] = y0;
                        a.q[(size_t)m * d + cb] = y1;
                    } else {
                        a.kc[slot + ca] = f32_to_bf16_bits(y0);
                        a.kc[slot + cb] = f32_to_bf16_bits(y1);
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------- many rows: what the projections above do in their epilogues
// Beyond fused_rows() the projections are GEMMs of their own (the LM head's kernels) with fp32 results `y`.
__global__ __launch_bounds__(kBlock) void k_body_add(size_t count4, float4* __restrict__ x, const float4* __restrict__ y) {
    const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= count4) return;
    const float4 a = x[i], b = y[i];
    x[i] = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

__global__ __launch_bounds__(kBlock) void k_body_silu_mul(int rows, int d_ff, const float* __restrict__ gu /* [rows, 2 d_ff] */,
                                                          uint16_t* __restrict__ act) {
    const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= (size_t)rows * d_ff) return;
    const size_t r = i / d_ff, f = i % d_ff;
    const float gte = gu[r * 2 * d_ff + f], up = gu[r * 2 * d_ff + d_ff + f];
    act[i] = f32_to_bf16_bits(gte / (1.f + __expf(-gte)) * up);
}

__global__ __launch_bounds__(kBlock) void k_body_rope(int d, int hd, int max_ctx, const float* __restrict__ qkv /* [rows,3d] */,
                                                      const double2* __restrict__ trig, const int32_t* __restrict__ ctx_len,
                                                      float* __restrict__ q, uint16_t* __restrict__ kc, uint16_t* __restrict__ vc) {
    const int r = blockIdx.x, half = hd / 2;
    const int pos = min(max(ctx_len[r], 0), max_ctx - 1);
    const size_t slot = ((size_t)r * max_ctx + pos) * d;
    for (int t = threadIdx.x; t < d / 2; t += kBlock) {
        const int i = t % half, ca = t / half * hd + i, cb = ca + half;
        const double2 cs = trig[(size_t)r * half + i];
        const float* y = qkv + (size_t)r * 3 * d;
        auto first = [&](const float* p) { return (float)((double)p[ca] * cs.x - (double)p[cb] * cs.y); };
        auto second = [&](const float* p) { return (float)((double)p[cb] * cs.x + (double)p[ca] * cs.y); };
        q[(size_t)r * d + ca] = first(y);
        q[(size_t)r * d + cb] = second(y);
        kc[slot + ca] = f32_to_bf16_bits(first(y + d));
        kc[slot + cb] = f32_to_bf16_bits(second(y + d));
        vc[slot + ca] = f32_to_bf16_bits(y[2 * d + ca]);
        vc[slot + cb] = f32_to_bf16_bits(y[2 * d + cb]);
    }
}

// ---------------------------------------------------------------- attention over the row's cache
// Grid (head, row, key range), four waves.  A key's (value's) head slice is hd contiguous bf16: LPK = hd / 8 lanes read it
// as 16-byte pieces, so one wave instruction fetches 64 / LPK whole slices.  Keys and values of a batch are requested
// together and one batch ahead of the one being used; every group of LPK lanes keeps a running maximum, sum and its 8
// dimensions of sum p v, and groups, then waves, are merged in a fixed order.  A row's keys are cut into gridDim.z ranges
// of equal length, whose sums the output projection merges.  HBM-bound at 64 rows (100 MB of keys and values in 20.3 us, 24.5 us
// with a pass over the keys, the softmax through LDS and a pass over the values); at few rows bound by how many compute
// units read (4 rows of 12 heads, 1250 positions: 33.5 us in one range, 6.5 us in eight).
constexpr int kAttnUnroll = 4;
template <int LPK>
__global__ __launch_bounds__(kBlock) void k_body_attn(int d, int max_ctx, const float* __restrict__ q, const int32_t* __restrict__ ctx_len,
                                                      const uint16_t* __restrict__ kc /* [rows,max_ctx,d] of this layer */,
                                                      const uint16_t* __restrict__ vc, uint16_t* __restrict__ att /* [rows,d]: one range */,
                                                      float* __restrict__ po, float* __restrict__ pml /* several ranges */) {
    constexpr int hd = LPK * 8, G = kWave / LPK;                          // G keys per wave instruction
    constexpr int kStride = kWavesPerBlock * G;                           // keys per workgroup instruction
    __shared__ float s_o[kWavesPerBlock][hd], s_m[kWavesPerBlock], s_l[kWavesPerBlock];
    const int hh = blockIdx.x, r = blockIdx.y, sp = blockIdx.z, S = gridDim.z, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int pos = ctx_len[r];
    pos = pos < 0 ? 0 : (pos >= max_ctx ? max_ctx - 1 : pos);
    const int T = pos + 1, chunk = ((T + S - 1) / S + kStride - 1) / kStride * kStride;
    const int t0 = sp * chunk, t1 = min(T, t0 + chunk);
    const int g = lane / LPK, c = lane % LPK;
    const uint16_t* Kr = kc + (size_t)r * max_ctx * d + hh * hd + c * 8;  // key t of this lane: Kr + t * d
    const uint16_t* Vr = vc + (size_t)r * max_ctx * d + hh * hd + c * 8;
    float qr[8];
    {
        const float scale = 1.44269504f / sqrtf((float)hd);               // scores in base 2
        const float4* qp = reinterpret_cast<const float4*>(q + (size_t)r * d + hh * hd + c * 8);
        const float4 a = qp[0], b = qp[1];
        qr[0] = a.x * scale; qr[1] = a.y * scale; qr[2] = a.z * scale; qr[3] = a.w * scale;
        qr[4] = b.x * scale; qr[5] = b.y * scale; qr[6] = b.z * scale; qr[7] = b.w * scale;
    }
    float m = -FLT_MAX, l = 0.f, o[8];        // not -inf: a range without keys subtracts it from itself; no finite score lies below
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = 0.f;
    if (t0 < t1) {
        const int mine = wave * G + g;
        u32x4b kw[kAttnUnroll], vw[kAttnUnroll], kn[kAttnUnroll], vn[kAttnUnroll];
        auto request = [&](u32x4b (&k4)[kAttnUnroll], u32x4b (&v4)[kAttnUnroll], int tb) {
#pragma unroll
            for (int u = 0; u < kAttnUnroll; ++u)                        // keys past the end re-read the last one
                k4[u] = *reinterpret_cast<const u32x4b*>(Kr + (size_t)min(tb + mine + u * kStride, t1 - 1) * d);
#pragma unroll
            for (int u = 0; u < kAttnUnroll; ++u)
                v4[u] = *reinterpret_cast<const u32x4b*>(Vr + (size_t)min(tb + mine + u * kStride, t1 - 1) * d);
        };
        request(kw, vw, t0);
        for (int tb = t0; tb < t1; tb += kStride * kAttnUnroll) {
            const bool more = tb + kStride * kAttnUnroll < t1;
            if (more) request(kn, vn, tb + kStride * kAttnUnroll);
            float sc[kAttnUnroll];
            float mn = m;
#pragma unroll
            for (int u = 0; u < kAttnUnroll; ++u) {
                float acc = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc += qr[2 * e] * __builtin_bit_cast(float, kw[u][e] << 16);
                    acc += qr[2 * e + 1] * __builtin_bit_cast(float, kw[u][e] & 0xffff0000u);
                }
                if (LPK > 1) acc += dpp_f32<kDppXor1>(acc);
                if (LPK > 2) acc += dpp_f32<kDppXor2>(acc);
                if (LPK > 4) acc += dpp_f32<kDppHalfMirror>(acc);
                if (LPK > 8) acc += dpp_f32<kDppMirror>(acc);
                sc[u] = (tb + mine + u * kStride < t1) ? acc : -INFINITY;
                mn = fmaxf(mn, sc[u]);
            }
            const float keep = __builtin_amdgcn_exp2f(m - mn);
            m = mn;
            l *= keep;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] *= keep;
#pragma unroll
            for (int u = 0; u < kAttnUnroll; ++u) {
                const float p = __builtin_amdgcn_exp2f(sc[u] - mn);
                l += p;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    o[2 * e] += p * __builtin_bit_cast(float, vw[u][e] << 16);
                    o[2 * e + 1] += p * __builtin_bit_cast(float, vw[u][e] & 0xffff0000u);
                }
            }
            if (more) {
#pragma unroll
                for (int u = 0; u < kAttnUnroll; ++u) { kw[u] = kn[u]; vw[u] = vn[u]; }
            }
        }
    }
    float mw = m;
#pragma unroll
    for (int off = LPK; off < kWave; off <<= 1) mw = fmaxf(mw, __shfl_xor(mw, off));
    const float keep = __builtin_amdgcn_exp2f(m - mw);
    l *= keep;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] *= keep;
#pragma unroll
    for (int off = LPK; off < kWave; off <<= 1) {
        l += __shfl_xor(l, off);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] += __shfl_xor(o[e], off);
    }
    if (lane < LPK) {
#pragma unroll
        for (int e = 0; e < 8; ++e) s_o[wave][lane * 8 + e] = o[e];
        if (lane == 0) { s_m[wave] = mw; s_l[wave] = l; }
    }
    __syncthreads();
    if (tid < hd) {
        const float M = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
        float sum = 0.f, L = 0.f;
#pragma unroll
        for (int w = 0; w < kWavesPerBlock; ++w) {
            const float f = __builtin_amdgcn_exp2f(s_m[w] - M);
            sum += s_o[w][tid] * f;
            L += s_l[w] * f;
        }
        if (S == 1) {
            att[(size_t)r * d + hh * hd + tid] = f32_to_bf16_bits(sum / L);
        } else {
            po[((size_t)sp * gridDim.y + r) * d + hh * hd + tid] = sum;
            if (tid == 0)
                *reinterpret_cast<float2*>(pml + (((size_t)r * gridDim.x + hh) * S + sp) * 2) = make_float2(M, L);
        }
    }
}

__global__ void k_body_rollback(int rows, int rows_per_seq, int gamma, const int32_t* __restrict__ ctx_base,
                                const int32_t* __restrict__ accept_len, int32_t* __restrict__ ctx_len) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= rows) return;
    const int k = accept_len[r / rows_per_seq];
    const int kept = (k + 1 < gamma) ? k + 1 : gamma;
    ctx_len[r] = ctx_base[r] + (kept < 0 ? 0 : kept);
}

// ---------------------------------------------------------------- host side
static size_t al256(size_t x) { return (x + 255) / 256 * 256; }

// Whether the fused projections run.  They read W once per 16 or 32 rows, a GEMM once per 64 to 256, but a GEMM writes and
// reads its result in fp32 and is two launches.  Two layers (d_ff = 4 d), fused / GEMM in us: d = 256 111 / 133 at 1024 rows,
// 183 / 172 at 2048; d = 768 182 / 195 at 384, 219 / 209 at 512; d = 1024 196 / 210 at 192, 232 / 217 at 256; d = 2048 293 / 407 at
// 128, 409 / 399 at 192, 949 / 514 at 512; one layer of d = 4096 (d_ff = 11264) 323 / 330 at 96, 397 / 348 at 128.
// Up to 64 rows the fused ones also keep the shorter chains of sums.
static bool fused_rows(int d, int rows) { return rows <= 64 || (long)rows * d <= 300 * 1024; }

// Whether a projection normalises its rows itself.  Each of its workgroups reads them whole, in fp32: beyond 1024 columns that
// leaves room for one block of 16 rows only, and W is read once per 16 rows.  Two layers of d = 2048 with the rows normalised
// in the projection / by a kernel of their own, in us: 100.5 / 103.0 at 1 row, 113.9 / 113.5 at 16, 146 / 119 at 17, 250 / 182 at
// 64; d = 1152 75.4 / 76.7 at 16, 84.9 / 81.7 at 17, 136 / 115 at 64.
static bool norm_in_projection(int d, int rows) { return d <= 1024 || (d <= 2048 && rows <= 16); }

// A projection [rows,K] x [N,K]^T as an LM head with vocabulary N, hidden size K, one draft and `rows` sequences.
static tabed_cfg gemm_cfg(int rows, int K, int N) {
    tabed_cfg c{};
    c.V = N; c.d = K; c.n = 1; c.B = rows; c.gamma = 1; c.h = 1; c.w_dtype = 1; c.distance = 0; c.policy = 0;
    c.tau_w = 1.f; c.eps = 1e-6f; c.seed = 0;
    return c;
}

// Key ranges a row's attention is cut into: enough for 768 workgroups (three per compute unit), at most 8, none shorter
// than 64 positions of a full cache; one where the output projection could not stage the merged rows in LDS.  Measured at
// 64 rows of 12 heads, 256 to 768 positions: attention 20.3 / 19.0 / 18.5 us with 1 / 2 / 4 ranges, but the projection that
// merges them 4.7 / 6.3 / 7.3 us.  4 rows of 12 heads, 600 to 1900 positions: 33 us with one range, 6.5 us with 8.
static int attn_splits(const tabed_body_cfg& c, int rows) {
    if (c.d > 1536 || !fused_rows(c.d, rows)) return 1;
    int S = 1;
    while (S < 8 && (long)rows * c.heads * S < 768 && c.max_ctx / (2 * S) >= 64) S *= 2;
    return S;
}

int body_route(const tabed_body_cfg& c, int rows) { return gang_applies(c, rows) ? 0 : attn_splits(c, rows); }

BodyLayout body_layout(const tabed_body_cfg& c, int rows) {
    BodyLayout L;
    const int act = (c.d > c.d_ff) ? c.d : c.d_ff;
    const size_t S = (size_t)attn_splits(c, rows);
    size_t off = 0;
    L.off_ctl = off;  off += kGangControlBytes;
    // (here, so that where its buffers are follows from the sizes that the control block remembers them by, which leave max_ctx out)
    L.off_gang = off; off = al256(off + (gang_applies(c, rows) ? gang_bytes(c, rows) : 0));
    L.off_x = off;    off = al256(off + sizeof(float) * (size_t)rows * c.d);
    L.off_q = off;    off = al256(off + sizeof(float) * (size_t)rows * c.d);
    L.off_trig = off; off = al256(off + sizeof(double2) * (size_t)rows * ((c.d / c.heads) / 2));
    L.off_hb = off;   off = al256(off + sizeof(uint16_t) * (size_t)rows * act);
    const bool many = !fused_rows(c.d, rows);
    L.off_hn = off;   off = al256(off + (many || !norm_in_projection(c.d, rows) ? sizeof(uint16_t) * (size_t)rows * c.d : 0));
    L.off_po = off;   off = al256(off + (S > 1 ? sizeof(float) * S * rows * c.d : 0));
    L.off_pml = off;  off = al256(off + (S > 1 ? sizeof(float) * 2 * S * rows * c.heads : 0));
    size_t gemm = 0;
    if (many)
        for (const auto& kn : {std::pair<int, int>{c.d, 3 * c.d}, {c.d, c.d}, {c.d, 2 * c.d_ff}, {c.d_ff, c.d}})
            gemm = std::max(gemm, ws_bytes_unpacked(gemm_cfg(rows, kn.first, kn.second)));
    L.off_y = off;    off = al256(off + (many ? sizeof(float) * (size_t)rows * std::max(3 * c.d, 2 * c.d_ff) : 0));
    L.off_gemm = off; off = al256(off + gemm);
    L.off_ones = off; off = al256(off + (many ? sizeof(float) * (size_t)rows : 0));
    L.total = off;
    return L;
}

// What steps of any number of rows up to `rows` need.  More rows need more, except that the one-launch step (up to 16 rows) has
// buffers that others have not, and that more rows have their keys in fewer ranges: each of these at the most rows that it occurs with.
size_t body_workspace_bytes(const tabed_body_cfg& c, int rows) {
    size_t most = 0;
    for (int r : {rows, 16, 767 / (4 * c.heads), 767 / (2 * c.heads), 767 / c.heads})
        if (r >= 1) most = std::max(most, body_layout(c, std::min(r, rows)).total);
    return most;
}

int validate_body_cfg(const tabed_body_cfg* c, int rows) {
    if (c == nullptr) return TABED_ENULL;
    if (c->layers < 1 || c->layers > TABED_BODY_MAX_LAYERS) return TABED_ERANGE;
    if (c->d < 8 || c->d % 8 != 0 || c->d_ff < 8 || c->d_ff % 8 != 0 || c->heads < 1 || c->d % c->heads != 0) return TABED_EINVAL;
    const int hd = c->d / c->heads;
    if (hd != 8 && hd != 16 && hd != 32 && hd != 64 && hd != 128) return TABED_EINVAL;
    if (c->V < 1 || c->max_ctx < 1 || c->max_ctx > 8192) return TABED_ERANGE;
    if (!(c->rope_theta > 0.f) || !(c->rms_eps > 0.f)) return TABED_EINVAL;
    if (rows < 1 || rows > 65535) return TABED_ERANGE;
    if (c->d > 8192 || 2 * c->d_ff > 262144) return TABED_ERANGE;
    return TABED_OK;
}

// All that a step expects to find is the one-launch step's control block, at the same place for all sizes.
hipError_t launch_body_init(const tabed_body_cfg& c, int rows, char* ws, hipStream_t s) { return launch_gang_init(ws + body_layout(c, rows).off_ctl, s); }

template <int NW, int MB, int G, int CI, int IN, int EPI>
static hipError_t launch_proj_t(int tiles, hipStream_t s, const ProjArgs& a) {
    constexpr int NB = (EPI == kEpiAdd) ? 1 : 2;
    constexpr size_t patches = (size_t)NW * (NB + (IN == kInBf16 ? MB : 0)) * kBodyPatch, results = sizeof(float) * NW * NB * MB * 16 * 20;
    auto lds = [&](int K) { return std::max(results, patches + ((IN == kInBf16) ? 0 : sizeof(uint16_t) * MB * 16 * (size_t)staged_row(K))); };
    static std::once_flag once;
    static hipError_t rc = hipSuccess;
    const size_t most = lds(IN == kInNorm ? CI * 256 : 1536);
    if (raise_lds_limit(&k_body_proj<NW, MB, G, CI, IN, EPI>, most, once, rc) != hipSuccess) return rc;
    ProfScope prof(TABED_K_BODY, s);
    launch(&prof, k_body_proj<NW, MB, G, CI, IN, EPI>, dim3(tiles, (a.M + MB * 16 - 1) / (MB * 16)), dim3(NW * 64), lds(a.K), s, a);
    return hipGetLastError();
}

// Waves per workgroup and k-blocks a wave requests together: four waves up to 1024 of contraction (eight for q/k/v: 7.2
// against 8.6 us at 64 rows), eight beyond, and as many requests as cover a wave's share where that is at most eight.  Two row
// blocks per workgroup, so that W is read half as often, where the tiles of one already fill the chip twice (once, for rows that
// are normalised here); with more than 48 k-blocks, whose W takes longest, where 192 workgroups are left (two layers of
// d = 2048, d_ff = 16384, 33 rows 264 us, 284 with one; d = 1024, d_ff = 4096, 64 rows, where 128 would be left, 84, 88 with two).
template <int IN, int EPI>
static hipError_t projection(const ProjArgs& a, int tiles, hipStream_t s) {
    const int mblocks = (a.M + 15) / 16;
    const int KB = (a.K + 63) / 64;
    const bool two = mblocks > 1 && (IN == kInNorm ? (long)tiles * mblocks >= 256
                                     : KB > 48     ? (long)tiles * ((mblocks + 1) / 2) >= 192
                                                   : (long)tiles * mblocks >= 512);
    if constexpr (IN == kInMerge) {
        return launch_proj_t<8, 1, 3, 1, IN, EPI>(tiles, s, a);
    } else if constexpr (IN == kInNorm) {
        if constexpr (EPI == kEpiRope) {                   // fewer workgroups than compute units: twice the waves in each
            if (a.K <= 768) return two ? launch_proj_t<8, 2, 2, 3, IN, EPI>(tiles, s, a) : launch_proj_t<8, 1, 2, 3, IN, EPI>(tiles, s, a);
            if (a.K <= 1024) return two ? launch_proj_t<8, 2, 2, 4, IN, EPI>(tiles, s, a) : launch_proj_t<8, 1, 2, 4, IN, EPI>(tiles, s, a);
        }
        if (a.K <= 768) return two ? launch_proj_t<4, 2, 3, 3, IN, EPI>(tiles, s, a) : launch_proj_t<4, 1, 3, 3, IN, EPI>(tiles, s, a);
        if (a.K <= 1024) return two ? launch_proj_t<4, 2, 4, 4, IN, EPI>(tiles, s, a) : launch_proj_t<4, 1, 4, 4, IN, EPI>(tiles, s, a);
        return launch_proj_t<8, 1, 4, 8, IN, EPI>(tiles, s, a);
    } else {
        if constexpr (EPI == kEpiAdd) {
            if (KB <= 12) return two ? launch_proj_t<4, 2, 3, 1, IN, EPI>(tiles, s, a) : launch_proj_t<4, 1, 3, 1, IN, EPI>(tiles, s, a);
            if (KB <= 16) return two ? launch_proj_t<4, 2, 4, 1, IN, EPI>(tiles, s, a) : launch_proj_t<4, 1, 4, 1, IN, EPI>(tiles, s, a);
            if (KB > 48) return two ? launch_proj_t<8, 2, 8, 1, IN, EPI>(tiles, s, a) : launch_proj_t<8, 1, 8, 1, IN, EPI>(tiles, s, a);
        }
        return two ? launch_proj_t<8, 2, 6, 1, IN, EPI>(tiles, s, a) : launch_proj_t<8, 1, 6, 1, IN, EPI>(tiles, s, a);
    }
}

static hipError_t launch_norm(const ProjArgs& a, uint16_t* out, int32_t* ctx_len_advance, hipStream_t s) {
    ProfScope prof(TABED_K_BODY, s);
    launch(&prof, k_body_norm, dim3(a.M), dim3(kBlock), 0, s, a.K, a.eps, static_cast<const float*>(a.x), a.g, out, ctx_len_advance);
    return hipGetLastError();
}

// The GEMM route of a projection: GEMM, then the epilogue as a kernel of its own.
template <int EPI>
static hipError_t gemm_projection(const ProjArgs& a, const uint16_t* X, char* ws, const BodyLayout& L, hipStream_t s) {
    const int N = (EPI == kEpiSilu) ? 2 * a.N : a.N;
    const tabed_cfg gc = gemm_cfg(a.M, a.K, N);
    float* y = reinterpret_cast<float*>(ws + L.off_y);
    const hipError_t e = launch_lmhead(gc, ws_layout(gc), ws + L.off_gemm, a.W, X, reinterpret_cast<const float*>(ws + L.off_ones), y, s,
                                       TABED_K_BODY);
    if (e != hipSuccess) return e;
    ProfScope prof(TABED_K_BODY, s);
    if (EPI == kEpiRope) {
        launch(&prof, k_body_rope, dim3(a.M), dim3(kBlock), 0, s, a.K, a.hd, a.max_ctx, static_cast<const float*>(y), a.trig, a.ctx_len, a.q,
               a.kc, a.vc);
    } else {
        const size_t count = (EPI == kEpiSilu) ? (size_t)a.M * a.N : (size_t)a.M * a.N / 4;
        const dim3 grid((unsigned)((count + kBlock - 1) / kBlock));
        if (EPI == kEpiSilu) launch(&prof, k_body_silu_mul, grid, dim3(kBlock), 0, s, a.M, a.N, static_cast<const float*>(y), a.act);
        else launch(&prof, k_body_add, grid, dim3(kBlock), 0, s, count, reinterpret_cast<float4*>(a.x), reinterpret_cast<const float4*>(y));
    }
    return hipGetLastError();
}

// RMSNorm + projection: in one launch where the projection normalises its rows itself.
template <int EPI>
static hipError_t norm_projection(ProjArgs a, uint16_t* hn, int tiles, char* ws, const BodyLayout& L, hipStream_t s) {
    const bool many = !fused_rows(a.K, a.M);
    if (!many && norm_in_projection(a.K, a.M)) return projection<kInNorm, EPI>(a, tiles, s);
    const hipError_t e = launch_norm(a, hn, nullptr, s);
    if (e != hipSuccess) return e;
    if (many) return gemm_projection<EPI>(a, hn, ws, L, s);
    a.X = hn;
    return projection<kInBf16, EPI>(a, tiles, s);
}

template <int LPK>
static void launch_attn(const ProfScope* prof, const tabed_body_cfg& c, int rows, int splits, const float* q, const int32_t* ctx_len,
                        const uint16_t* kc, const uint16_t* vc, uint16_t* att, float* po, float* pml, hipStream_t s) {
    launch(prof, k_body_attn<LPK>, dim3(c.heads, rows, splits), dim3(kBlock), 0, s, c.d, c.max_ctx, q, ctx_len, kc, vc, att, po, pml);
}

hipError_t launch_body_step(const tabed_body_cfg& c, const tabed_body_weights& w, char* ws, int rows,
                            const int32_t* token_src, int token_stride, int rows_per_token, int32_t* ctx_len,
                            uint16_t* kcache, uint16_t* vcache, uint16_t* H, hipStream_t s, int late_from, int absent) {
    const BodyLayout L = body_layout(c, rows);
    if (gang_applies(c, rows))
        return launch_gang(c, w, ws + L.off_ctl, ws + L.off_gang, rows, token_src, token_stride, rows_per_token, ctx_len, kcache, vcache, H, s,
                           late_from, absent);
    uint16_t* hb = reinterpret_cast<uint16_t*>(ws + L.off_hb);
    float* po = reinterpret_cast<float*>(ws + L.off_po);
    float* pml = reinterpret_cast<float*>(ws + L.off_pml);
    const int d = c.d, hd = c.d / c.heads, splits = attn_splits(c, rows);
    const bool many = !fused_rows(c.d, rows);
    uint16_t* hn = reinterpret_cast<uint16_t*>(ws + L.off_hn);
    ProjArgs base{};
    base.M = rows; base.eps = c.rms_eps; base.hd = hd; base.max_ctx = c.max_ctx;
    base.ctx_len = ctx_len; base.splits = splits; base.po = po; base.pml = pml;
    base.x = reinterpret_cast<float*>(ws + L.off_x);
    base.q = reinterpret_cast<float*>(ws + L.off_q);
    base.X = hb; base.act = hb;
    double2* trig = reinterpret_cast<double2*>(ws + L.off_trig);
    base.trig = trig;
    hipError_t e;
    {
        ProfScope prof(TABED_K_BODY, s);
        launch(&prof, k_body_embed, dim3(rows), dim3(kBlock), 0, s, d, c.V, token_src, token_stride, rows_per_token,
               static_cast<const uint16_t*>(w.embed), base.x, static_cast<const int32_t*>(ctx_len), c.max_ctx, hd,
               std::log2((double)c.rope_theta), trig, gang_key(ws + L.off_ctl), many ? reinterpret_cast<float*>(ws + L.off_ones) : nullptr);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    for (int l = 0; l < c.layers; ++l) {
        const size_t layer_off = (size_t)l * rows * c.max_ctx * d;
        ProjArgs a = base;
        a.kc = kcache + layer_off; a.vc = vcache + layer_off;
        a.W = static_cast<const uint16_t*>(w.wqkv[l]); a.N = 3 * d; a.K = d; a.g = w.g_attn[l];
        if ((e = norm_projection<kEpiRope>(a, hn, 3 * ((d + 31) / 32), ws, L, s)) != hipSuccess) return e;
        {
            ProfScope prof(TABED_K_BODY, s);
            switch (hd) {
                case 8: launch_attn<1>(&prof, c, rows, splits, a.q, ctx_len, a.kc, a.vc, hb, po, pml, s); break;
                case 16: launch_attn<2>(&prof, c, rows, splits, a.q, ctx_len, a.kc, a.vc, hb, po, pml, s); break;
                case 32: launch_attn<4>(&prof, c, rows, splits, a.q, ctx_len, a.kc, a.vc, hb, po, pml, s); break;
                case 64: launch_attn<8>(&prof, c, rows, splits, a.q, ctx_len, a.kc, a.vc, hb, po, pml, s); break;
                case 128: launch_attn<16>(&prof, c, rows, splits, a.q, ctx_len, a.kc, a.vc, hb, po, pml, s); break;
                default: return hipErrorInvalidValue;
            }
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        a = base;
        a.W = static_cast<const uint16_t*>(w.wo[l]); a.N = d; a.K = d;
        if (many) e = gemm_projection<kEpiAdd>(a, hb, ws, L, s);
        else if (splits > 1) e = projection<kInMerge, kEpiAdd>(a, (d + 15) / 16, s);
        else e = projection<kInBf16, kEpiAdd>(a, (d + 15) / 16, s);
        if (e != hipSuccess) return e;
        a = base;
        a.W = static_cast<const uint16_t*>(w.wgu[l]); a.N = c.d_ff; a.K = d; a.g = w.g_mlp[l];
        if ((e = norm_projection<kEpiSilu>(a, hn, (c.d_ff + 15) / 16, ws, L, s)) != hipSuccess) return e;
        a = base;
        a.W = static_cast<const uint16_t*>(w.wdown[l]); a.N = d; a.K = c.d_ff;
        e = many ? gemm_projection<kEpiAdd>(a, hb, ws, L, s) : projection<kInBf16, kEpiAdd>(a, (d + 15) / 16, s);
        if (e != hipSuccess) return e;
    }
    ProjArgs a = base;
    a.K = d; a.g = w.g_final;
    return launch_norm(a, H, ctx_len, s);
}

hipError_t launch_body_rollback(int rows, int rows_per_seq, int gamma, const int32_t* ctx_base, const int32_t* accept_len,
                                int32_t* ctx_len, hipStream_t s) {
    launch(nullptr, k_body_rollback, dim3((rows + 255) / 256), dim3(256), 0, s, rows, rows_per_seq, gamma, ctx_base, accept_len,
           ctx_len);
    return hipGetLastError();
}

}  // namespace tabed
