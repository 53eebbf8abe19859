// LM head of the n batched drafts (Alg. 1 (draft forward), last layer of the shared draft model):
//   L[r, v] = sum_k H[r, k] * W[v, k],   r = b*n + j  (M = n*B rows),
// with the first half of the per-draft softmax fused into the epilogue: for every row and every 32-wide
// vocabulary tile the kernel also writes  pm = max_v s(v)  and  ps = sum_v exp(s(v) - pm),  s = L / T_b.
// gfx950: bf16 operands go through v_mfma_f32_32x32x16_bf16, in the W-streaming kernel v_mfma_f32_16x16x32_bf16 (fp32
// accumulate); fp32 operands (the tiny correctness configuration) use plain FMAs.
#include <hip/hip_bf16.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "device_utils.h"
#include "internal.h"

namespace tabed {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // four floats that are only 4-byte aligned

__device__ __forceinline__ float inv_temperature(float T) { return (T > 0.f) ? 1.f / T : 1.f; }
__device__ __forceinline__ float row_inv_temperature(const float* temperature, int row, int n) { return inv_temperature(temperature[row / n]); }
// row / n for row < 65536 without an integer division: (row + 1/2) / n is at least 1 / 32 away from an integer (n <= 16),
// far more than the error of the reciprocal.
__device__ __forceinline__ int sequence_of(int row, int n) { return (int)(((float)row + 0.5f) * __builtin_amdgcn_rcpf((float)n)); }

// Reductions over the 32 lanes that share lane/32 (xor offsets < 32 never leave the half-wave).
__device__ __forceinline__ float half_max(float v) {
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ float half_sum(float v) {
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Four logits of a row, past L2 or, of more than 64 rows, through it.  Rows whose 64-byte sectors are shared by neighbouring tiles go through L2, which puts
// the sectors together, where there are so many logits that storing parts of sectors is what takes the time.  Draft steps in us,
// through / past L2: V = 100003, 255 rows, d = 1024 133 / 155, 128 rows, d = 640 68.8 / 78.4, V = 50004, 96 rows, d = 768 35.4 / 36.2,
// V = 32001, 480 rows, d = 72 49.3 / 59.9; but below 16 MB of logits, most of which would be left to the write-back at the end, V = 20001,
// 80 rows, d = 2048 36.1 / 31.3, V = 30001, 120 rows, d = 1160 36.8 / 35.9; up to 64 rows, whose stores go out beside the stream of W,
// V = 100003 60.3 / 57.8 at 64 rows, 52.4 / 50.6 at 32; and with whole sectors, V = 100000, 128 rows 61.9 / 54.9.
// The exception: W of about the last-level cache's size (256 MB) stays there from one draft step to the next, unless logits stored
// through L2 take its place, which costs more than the sectors where the logits are few beside W (the ratio of their bytes is 2 M / d).
// Steps back to back on the same buffers, through / past L2, us.  128 rows, d = 3000, W of 240 MB, V = 40001 98.6 / 75.2, 40008 96.8 / 74.3; of 205 MB,
// 34168 73.6 / 73.1, of 320 MB, 53329 104.7 / 107.5.  d = 1328, 225 MB, V = 84708 85.8 / 80.6, with 256 rows 130.6 / 135.8, V = 84705 86.5 / 83.9,
// 132.2 / 142.2; 205 MB 67.8 / 76.9.  66 rows, d = 520, 255 MB, V = 245192 112.8 / 100.5, 128 rows 142.5 / 138.9.  Whole lines lose less, later:
// 128 rows, d = 2048, 240 MB 54.5 / 56.8, 270 MB, V = 65908 98.8 / 91.7, 320 MB 119.4 / 126.7; 96 rows, d = 896, 255 MB 82.7 / 83.9.
static bool past_l2(int V, int d, int M) {
    if ((V & 15) == 0 || (long)M * V < (4l << 20)) return true;
    const bool lines = d % 64 == 0;
    const long w = 2l * V * d;
    return w > (lines ? 250000000l : 222000000l) && w < (lines ? 300000000l : 278000000l) && 2l * d >= (lines ? 28l : (V & 3) ? 22l : 15l) * M;
}
// (An instance each: a choice at run time between the two stores becomes one that goes through L2.)
template <bool PAST>
__device__ __forceinline__ void store_logits(float* p, f32x4u x) {
    if constexpr (PAST) __builtin_nontemporal_store(x, reinterpret_cast<f32x4u*>(p));
    else *reinterpret_cast<f32x4u*>(p) = x;
}

constexpr int kPatchBytes = 32 * 144;                  // LDS in which a wave turns 32 rows of 32 floats

// Epilogue of one 32x32 accumulator tile held TRANSPOSED: lane holds result row m_base + lane % 32 and the 16
// vocabulary entries v_base + 8*(r/4) + 4*(lane/32) + r%4.  The softmax partials of a row are then a
// 16-value in-register reduction plus one exchange between the two half-waves, and every lane stores four
// runs of four consecutive logits.  inv_t[m] = 1/T of row m (LDS table).  With `pstage` the partials go to an
// LDS table instead, from which the caller writes a workgroup's four tiles of a row as one 16-byte store.
template <bool PAST = true>
__device__ __forceinline__ void store_tile_32x32_t(const f32x16& acc, int m_base, int v_base, int M, int V, int NT,
                                                   const float* inv_t, float* __restrict__ L,
                                                   float* __restrict__ pm, float* __restrict__ ps,
                                                   unsigned char* tpatch, float* pstage = nullptr, int pslot = 0) {
    if (v_base >= V) return;
    const int lane = threadIdx.x & 63;
    const int col = lane & 31, half = lane >> 5;
    const int m = m_base + col;
    const bool live = (m < M);
    const float it = live ? inv_t[m] : 1.f;
    const bool full = v_base + 32 <= V;            // uniform: only the last tile of a row is ragged
    float x[16];
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = acc[r];            // (rows past the end: computed, not stored)
    if (!full) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (v_base + 8 * (r / 4) + 4 * half + (r % 4) >= V) x[r] = -INFINITY;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, x[r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    mx = (mx > -INFINITY) ? mx * it : mx;                  // (the largest product: 1 / T is positive and rounding keeps the order)
    const float base = (mx > -INFINITY) ? mx : 0.f;        // a tile of -inf sums to 0
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) sum += __expf(fmaf(x[r], it, -base));
    if (__any(sum != sum)) {                               // a NaN logit has no mass and does not take the tile's with it
        sum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += (x[r] * it > -INFINITY) ? __expf(fmaf(x[r], it, -mx)) : 0.f;
    }
    sum += __shfl_xor(sum, 32);
    if (live && half == 0) {
        if (pstage != nullptr) {                    // collected per workgroup: [array][row][tile of the group]
            pstage[(0 * 64 + m) * 4 + pslot] = mx;
            pstage[(1 * 64 + m) * 4 + pslot] = sum;
        } else {
            pm[(size_t)m * NT + v_base / kTileV] = mx;
            ps[(size_t)m * NT + v_base / kTileV] = sum;
        }
    }
    if (full) {
        // Full tile: turn the block through the wave's LDS patch ([32 rows][32 v] floats, 144-byte rows) so
        // that 8 lanes store one whole 128-byte line of a row, and stream it past L2: the logits are next
        // read tens of megabytes later, and full-line streaming stores measured 1.9 us faster per launch
        // than leaving 8 MB of dirty partial lines to the end-of-kernel write-back.
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<float4*>(tpatch + col * 144 + (8 * g + 4 * half) * 4) =
                make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int mr = 8 * i + (lane >> 3), q = lane & 7;
            const float4 val = *reinterpret_cast<const float4*>(tpatch + mr * 144 + q * 16);
            if (m_base + mr < M)                   // (rows of an odd vocabulary are only 4-byte aligned)
                store_logits<PAST>(L + (size_t)(m_base + mr) * V + v_base + 4 * q, f32x4u{val.x, val.y, val.z, val.w});
        }
        return;
    }
    if (!live) return;
    float* row = L + (size_t)m * V;                // ragged last tile: element-wise
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int v = v_base + 8 * g + 4 * half + e;
            if (v < V) row[v] = acc[4 * g + e];
        }
}

// The other half-wave's value beside this one's: {lanes 0-31, lanes 0-31} and {lanes 32-63, lanes 32-63}.
__device__ __forceinline__ float2 both_halves(float v) {
    const auto p = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
    return make_float2(__builtin_bit_cast(float, (unsigned)p[0]), __builtin_bit_cast(float, (unsigned)p[1]));
}

// Epilogue of a wave's TV x TM accumulator tiles, none of which reaches past the vocabulary: the values, the operations and their
// order are those of store_tile_32x32_t.  The row tiles of a vocabulary tile go through each phase side by side, so that none waits for
// its own chain (maximum, exchange, exponentials, exchange), and the partials of the workgroup's rows are collected in LDS
// (part: [row][kPT tiles] maxima, kPS floats on the sums), from where a row's are stored 16 bytes at a time: a store of their own for
// every tile and row was two of three memory requests of the epilogue.
// rows: how many rows of the wave's block exist; patch: two of kPatchBytes.
template <bool PAST, int TV, int TM, int kPT, int kPS>
__device__ __forceinline__ void store_full_tiles(const f32x16 (&acc)[TV][TM], int rows, const float* s_it, float* part, float* L /* row, entry 0 of the block */,
                                                 int V, unsigned char* patch) {
    const int lane = threadIdx.x & 63, col = lane & 31, half = lane >> 5;
    float it[TM];
#pragma unroll
    for (int b = 0; b < TM; ++b) it[b] = s_it[b * 32 + col];
#pragma unroll
    for (int a = 0; a < TV; ++a) {
        float mx[TM], base[TM], sum[TM];
#pragma unroll
        for (int b = 0; b < TM; ++b) {
            mx[b] = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) mx[b] = fmaxf(mx[b], acc[a][b][r]);
        }
#pragma unroll
        for (int b = 0; b < TM; ++b) {
            const float2 h = both_halves(mx[b]);
            mx[b] = fmaxf(h.x, h.y);
            mx[b] = (mx[b] > -INFINITY) ? mx[b] * it[b] : mx[b];
            base[b] = (mx[b] > -INFINITY) ? mx[b] : 0.f;
            sum[b] = 0.f;
        }
#pragma unroll
        for (int b = 0; b < TM; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[b] += __expf(fmaf(acc[a][b][r], it[b], -base[b]));
        bool nan = false;
#pragma unroll
        for (int b = 0; b < TM; ++b) nan = nan || sum[b] != sum[b];
        if (__any(nan)) {                                  // a NaN logit has no mass and does not take the tile's with it
#pragma unroll
            for (int b = 0; b < TM; ++b) {
                if (!__any(sum[b] != sum[b])) continue;    // (tile by tile, as store_tile_32x32_t decides)
                sum[b] = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    sum[b] += (acc[a][b][r] * it[b] > -INFINITY) ? __expf(fmaf(acc[a][b][r], it[b], -mx[b])) : 0.f;
                }
            }
        }
#pragma unroll
        for (int b = 0; b < TM; ++b) {
            const float2 h = both_halves(sum[b]);
            if (half == 0) {
                part[(b * 32 + col) * kPT + a] = mx[b];
                part[(b * 32 + col) * kPT + a + kPS] = h.x + h.y;
            }
        }
#pragma unroll
        for (int b = 0; b < TM; ++b) {
            if (b * 32 >= rows) continue;                  // uniform
            unsigned char* const tp = patch + (b & 1) * kPatchBytes;
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4*>(tp + col * 144 + (8 * g + 4 * half) * 4) =
                    make_float4(acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2], acc[a][b][4 * g + 3]);
            const int q = lane & 7;
            float* const out = L + (size_t)(b * 32 + (lane >> 3)) * V + a * 32 + 4 * q;
            float4 val[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) val[i] = *reinterpret_cast<const float4*>(tp + (8 * i + (lane >> 3)) * 144 + q * 16);
            auto store = [&](int i) {
                store_logits<PAST>(out + (size_t)(8 * i) * V, f32x4u{val[i].x, val[i].y, val[i].z, val[i].w});
            };
            if ((b + 1) * 32 <= rows) {                    // uniform
#pragma unroll
                for (int i = 0; i < 4; ++i) store(i);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (b * 32 + 8 * i + (lane >> 3) < rows) store(i);
            }
        }
    }
}

// ---------------------------------------------------------------- bf16, up to 64 rows, d = 512, 768 or 896: W-streaming kernel
// With n*B <= 64 rows the GEMM moves 2*d bytes of W per n*B*2*d flops: it is bound by streaming W from HBM
// once, not by the matrix cores.  Design:
//   * 8 waves per workgroup, one workgroup per compute unit.  All of H (<= 64 x d bf16) is staged once into
//     LDS (rows padded by 16 bytes, so the 16-byte operand reads of 16 consecutive rows hit distinct banks).
//   * A pair of waves owns one 32-row vocabulary tile; each wave of the pair takes one half of K and streams
//     it k-block by k-block (32 rows x 128 bytes, coalesced 16-byte loads: 8 lanes cover one row's 128 bytes),
//     three k-blocks ahead of the one being multiplied.  W is read exactly once; no wave shares W with another.
//   * The MFMA wants "lane = vocabulary row, 8 consecutive k": each k-block goes through a wave-private
//     32 x 144-byte LDS patch that only re-maps lanes (write coalesced layout, read operand layout); LDS ops of
//     one wave execute in order, so the patch needs no barrier.
//   * W is the MFMA's row operand, so the accumulator is [vocabulary][result row]: the softmax partials of a
//     row are an in-register reduction plus one half-wave exchange.
//   * The two K-halves meet through the same patches (LDS-only barriers), each wave finishing one 32-row
//     block of the 64 x 32 result: logits (turned through the patch once more, stored as whole 128-byte lines
//     past L2) + softmax partials of the tile.
// KH = k-blocks (of 64) per wave = d / 128; MT = 32-row blocks of M.
constexpr int kSkinnyWaves = 8;
constexpr int kSkinnyThreads = kSkinnyWaves * 64;

template <int KH, int MT>
__global__ __launch_bounds__(kSkinnyThreads) void k_lmhead_skinny(int M, int V, int n, int NT, int num_tiles,
                                                                  const uint16_t* __restrict__ W,
                                                                  const uint16_t* __restrict__ H,
                                                                  const float* __restrict__ temperature,
                                                                  float* __restrict__ L, float* __restrict__ pm,
                                                                  float* __restrict__ ps) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ float s_invt[64];
    __shared__ __attribute__((aligned(16))) float s_pstage[2 * 64 * 4];   // softmax partials of the group's 4 tiles
    constexpr int d = KH * 128;
    constexpr int CH = d / 8;                       // 16-byte chunks per row of H / W
    constexpr int HROW = CH * 16 + 16;              // padded LDS row of H in bytes
    unsigned char* const ldsH = lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int pair = wave & 3, khalf = wave >> 2;
    unsigned char* const patch = lds + MT * 32 * HROW + wave * kPatchBytes;
    unsigned char* const partner_patch = lds + MT * 32 * HROW + (wave ^ 4) * kPatchBytes;
    const int nn = lane & 31, half = lane >> 5;
    // requested here, used after the loads below
    const float my_temp = temperature[sequence_of(min(tid, M - 1), n)];

    // ---- request H first (it must land before any MFMA)
    u32x4 hreg[MT * KH];
#pragma unroll
    for (int q = 0; q < MT * KH; ++q) {
        // rows >= M are clamped, not zeroed: their results are never stored
        const int p = tid + q * kSkinnyThreads, row = min(p / CH, M - 1), c = p % CH;
        hreg[q] = *reinterpret_cast<const u32x4*>(H + (size_t)row * d + c * 8);
    }
    const int lrow = lane >> 3, lchunk = lane & 7;  // coalesced load layout: instruction i covers rows 8i..8i+7
    u32x4 wreg[KH][4];
    // Requests of one k-block (4 coalesced 16-byte loads per lane).  Vocabulary rows >= V (ragged last tile,
    // idle pair of the last group) are clamped to row V-1: the epilogue masks them, so no load is predicated.
    // (element offsets from W, not pointers: a pointer carried in an array degrades to a flat address and
    // flat loads also count as LDS traffic, which would stall every LDS read behind them)
    auto aim_tile = [&](size_t (&off)[4], int tile) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int v = min(tile * 32 + 8 * i + lrow, V - 1);
            off[i] = (size_t)v * d + (size_t)khalf * (KH * 64) + lchunk * 8;
        }
    };
    auto request_kblock = [&](const size_t (&off)[4], int kb) {
#pragma unroll
        for (int i = 0; i < 4; ++i) wreg[kb][i] = *reinterpret_cast<const u32x4*>(W + off[i] + kb * 64);
    };
    // Only the first kPF k-blocks of W are requested before H has landed.  Measured on MI355X: a compute unit
    // accepts a bounded number of outstanding requests, so issuing a whole half-tile takes about as long as
    // streaming it, and with all of W queued behind them the H loads came back ~5 us late (nothing can start
    // without H).  With kPF k-blocks queued H lands at ~1.7 us and the first W data follows at once; the rest
    // of W is requested k-block by k-block, kPF ahead of the one being multiplied.
    constexpr int kPF = (KH < 3) ? KH : 3;
    size_t src[4];                                 // the tile whose k-blocks are being requested
    aim_tile(src, blockIdx.x * 4 + pair);
#pragma unroll
    for (int kb = 0; kb < kPF; ++kb) request_kblock(src, kb);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < MT * KH; ++q) {
        const int p = tid + q * kSkinnyThreads, row = p / CH, c = p % CH;
        *reinterpret_cast<u32x4*>(ldsH + row * HROW + c * 16) = hreg[q];
    }
    if (tid < M) s_invt[tid] = inv_temperature(my_temp);
    lds_barrier();                                 // also publishes s_invt

    for (int g = blockIdx.x;; g += gridDim.x) {    // tile group g = 4 tiles, one per wave pair; trip count is
        const int this_tile = g * 4 + pair;        // uniform over the workgroup (barriers inside)
        f32x16 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mt][r] = 0.f;
        const bool more = ((g + (int)gridDim.x) * 4 < num_tiles);   // this workgroup has another tile group
        size_t nsrc[4];
        aim_tile(nsrc, more ? this_tile + (int)gridDim.x * 4 : this_tile);
#pragma unroll
        for (int kb = 0; kb < KH; ++kb) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<u32x4*>(patch + (8 * i + lrow) * 144 + lchunk * 16) = wreg[kb][i];
            // the registers of k-block kb are free again: request the k-block kPF ahead (of this tile, or of
            // the workgroup's next tile once this one is fully requested)
            __builtin_amdgcn_sched_barrier(0);
            if (kb + kPF < KH) request_kblock(src, kb + kPF);
            else if (more) request_kblock(nsrc, kb + kPF - KH);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const bf16x8 bv = *reinterpret_cast<const bf16x8*>(patch + nn * 144 + (2 * ks + half) * 16);
                const int hc = (khalf * KH + kb) * 8 + 2 * ks + half;       // chunk index inside H's row
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const bf16x8 av = *reinterpret_cast<const bf16x8*>(ldsH + (mt * 32 + nn) * HROW + hc * 16);
                    // W fragment as the row operand: the accumulator comes out as [vocabulary][result row]
                    acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv, av, acc[mt], 0, 0, 0);
                }
            }
        }

        // ---- the two K-halves meet: each wave hands the partner the 32-row block the partner finishes
        //      (MT == 2: wave khalf finishes block khalf; MT == 1: the khalf == 0 wave finishes block 0)
        f32x16 fin = acc[0], giv = acc[MT - 1];
        if (MT == 2 && khalf == 1) { fin = acc[MT - 1]; giv = acc[0]; }
        if (MT == 2 || khalf == 1) {
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<float4*>(patch + g * 1024 + lane * 16) =
                    make_float4(giv[4 * g], giv[4 * g + 1], giv[4 * g + 2], giv[4 * g + 3]);
        }
        lds_barrier();
        if (MT == 2 || khalf == 0) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 o = *reinterpret_cast<const float4*>(partner_patch + g * 1024 + lane * 16);
                fin[4 * g] += o.x; fin[4 * g + 1] += o.y; fin[4 * g + 2] += o.z; fin[4 * g + 3] += o.w;
            }
        }
        lds_barrier();                                 // both patches of the pair are read: they may be reused
        if ((MT == 2 || khalf == 0) && this_tile < num_tiles)
            store_tile_32x32_t(fin, (MT == 2) ? khalf * 32 : 0, this_tile * 32, M, V, NT, s_invt, L, pm, ps, patch, s_pstage, pair);
        // the four tiles of this group sit side by side in a row of the partial tables: 16 bytes per row
        lds_barrier();
        if (tid < 128 && (tid & 63) < M) {
            const int arr = tid >> 6, row = tid & 63, t0 = g * 4;
            float* dst = (arr == 0 ? pm : ps) + (size_t)row * NT + t0;
            const float* srcp = s_pstage + (arr * 64 + row) * 4;
            if ((NT & 3) == 0 && t0 + 3 < NT) *reinterpret_cast<float4*>(dst) = *reinterpret_cast<const float4*>(srcp);
            else for (int q = 0; q < 4; ++q) if (t0 + q < NT) dst[q] = srcp[q];
        }
        if (!more) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) src[i] = nsrc[i];
    }
}

// ---------------------------------------------------------------- bf16, skinny M, larger hidden sizes
// Same design as k_lmhead_skinny for hidden sizes whose H (64 x d) does not fit LDS: K is walked in chunks of
// KH*128, and LDS holds one chunk of H at a time.  The next chunk of H is requested into registers at the
// start of a chunk's k-loop and written to LDS between two LDS-only barriers at its end; the W request
// stream (kPF k-blocks ahead) runs straight across chunk boundaries.  d = nchunks * KH * 128.
template <int KH, int MT>
__global__ __launch_bounds__(kSkinnyThreads) void k_lmhead_skinny_kc(int M, int V, int n, int NT, int num_tiles,
                                                                     int nchunks,
                                                                     const uint16_t* __restrict__ W,
                                                                     const uint16_t* __restrict__ H,
                                                                     const float* __restrict__ temperature,
                                                                     float* __restrict__ L, float* __restrict__ pm,
                                                                     float* __restrict__ ps) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ float s_invt[64];
    __shared__ __attribute__((aligned(16))) float s_pstage[2 * 64 * 4];   // softmax partials of the group's 4 tiles
    constexpr int DC = KH * 128;                    // k per chunk
    constexpr int CH = DC / 8;                      // 16-byte pieces per row of one H chunk
    constexpr int HROW = CH * 16 + 16;              // padded LDS row of H in bytes
    const int d = nchunks * DC;
    unsigned char* const ldsH = lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int pair = wave & 3, khalf = wave >> 2;
    unsigned char* const patch = lds + MT * 32 * HROW + wave * kPatchBytes;
    unsigned char* const partner_patch = lds + MT * 32 * HROW + (wave ^ 4) * kPatchBytes;
    const int nn = lane & 31, half = lane >> 5;
    const float my_temp = temperature[sequence_of(min(tid, M - 1), n)];   // used after the requests below

    u32x4 hreg[MT * KH];
    auto request_h = [&](int chunk) {               // rows >= M are clamped: their results are never stored
#pragma unroll
        for (int q = 0; q < MT * KH; ++q) {
            const int p = tid + q * kSkinnyThreads, row = min(p / CH, M - 1), c = p % CH;
            hreg[q] = *reinterpret_cast<const u32x4*>(H + (size_t)row * d + (size_t)chunk * DC + c * 8);
        }
    };
    auto write_h = [&]() {
#pragma unroll
        for (int q = 0; q < MT * KH; ++q) {
            const int p = tid + q * kSkinnyThreads, row = p / CH, c = p % CH;
            *reinterpret_cast<u32x4*>(ldsH + row * HROW + c * 16) = hreg[q];
        }
    };
    const int lrow = lane >> 3, lchunk = lane & 7;
    u32x4 wreg[KH][4];
    auto aim_tile = [&](size_t (&off)[4], int tile) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int v = min(tile * 32 + 8 * i + lrow, V - 1);
            off[i] = (size_t)v * d + (size_t)khalf * (KH * 64) + lchunk * 8;
        }
    };
    auto request_kblock = [&](const size_t (&off)[4], int chunk, int kb) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            wreg[kb][i] = *reinterpret_cast<const u32x4*>(W + off[i] + (size_t)chunk * DC + kb * 64);
    };
    constexpr int kPF = 3;                          // KH >= 4 here
    request_h(0);
    size_t src[4];
    aim_tile(src, blockIdx.x * 4 + pair);
#pragma unroll
    for (int kb = 0; kb < kPF; ++kb) request_kblock(src, 0, kb);
    __builtin_amdgcn_sched_barrier(0);
    write_h();
    if (tid < M) s_invt[tid] = inv_temperature(my_temp);
    lds_barrier();                                  // also publishes s_invt

    for (int g = blockIdx.x;; g += gridDim.x) {
        const int this_tile = g * 4 + pair;
        f32x16 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mt][r] = 0.f;
        const bool more = ((g + (int)gridDim.x) * 4 < num_tiles);
        size_t nsrc[4];
        aim_tile(nsrc, more ? this_tile + (int)gridDim.x * 4 : this_tile);
        for (int chunk = 0; chunk < nchunks; ++chunk) {
            const bool last_chunk = (chunk + 1 == nchunks);
            const bool h_next = !last_chunk || more;  // another chunk of H follows (of this tile or the next)
            if (h_next) request_h(last_chunk ? 0 : chunk + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kb = 0; kb < KH; ++kb) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    *reinterpret_cast<u32x4*>(patch + (8 * i + lrow) * 144 + lchunk * 16) = wreg[kb][i];
                __builtin_amdgcn_sched_barrier(0);
                if (kb + kPF < KH) request_kblock(src, chunk, kb + kPF);
                else if (!last_chunk) request_kblock(src, chunk + 1, kb + kPF - KH);
                else if (more) request_kblock(nsrc, 0, kb + kPF - KH);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const bf16x8 bv = *reinterpret_cast<const bf16x8*>(patch + nn * 144 + (2 * ks + half) * 16);
                    const int hc = (khalf * KH + kb) * 8 + 2 * ks + half;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const bf16x8 av = *reinterpret_cast<const bf16x8*>(ldsH + (mt * 32 + nn) * HROW + hc * 16);
                        acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bv, av, acc[mt], 0, 0, 0);
                    }
                }
            }
            if (h_next) {
                lds_barrier();                      // every wave is done with this chunk of H
                write_h();
                lds_barrier();
            }
        }

        f32x16 fin = acc[0], giv = acc[MT - 1];
        if (MT == 2 && khalf == 1) { fin = acc[MT - 1]; giv = acc[0]; }
        if (MT == 2 || khalf == 1) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4*>(patch + q * 1024 + lane * 16) =
                    make_float4(giv[4 * q], giv[4 * q + 1], giv[4 * q + 2], giv[4 * q + 3]);
        }
        lds_barrier();
        if (MT == 2 || khalf == 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 o = *reinterpret_cast<const float4*>(partner_patch + q * 1024 + lane * 16);
                fin[4 * q] += o.x; fin[4 * q + 1] += o.y; fin[4 * q + 2] += o.z; fin[4 * q + 3] += o.w;
            }
        }
        lds_barrier();
        if ((MT == 2 || khalf == 0) && this_tile < num_tiles)
            store_tile_32x32_t(fin, (MT == 2) ? khalf * 32 : 0, this_tile * 32, M, V, NT, s_invt, L, pm, ps, patch, s_pstage, pair);
        // the four tiles of this group sit side by side in a row of the partial tables: 16 bytes per row
        lds_barrier();
        if (tid < 128 && (tid & 63) < M) {
            const int arr = tid >> 6, row = tid & 63, t0 = g * 4;
            float* dst = (arr == 0 ? pm : ps) + (size_t)row * NT + t0;
            const float* srcp = s_pstage + (arr * 64 + row) * 4;
            if ((NT & 3) == 0 && t0 + 3 < NT) *reinterpret_cast<float4*>(dst) = *reinterpret_cast<const float4*>(srcp);
            else for (int q = 0; q < 4; ++q) if (t0 + q < NT) dst[q] = srcp[q];
        }
        if (!more) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) src[i] = nsrc[i];
    }
}

// ---------------------------------------------------------------- bf16, up to 64 rows, any hidden size: W-streaming kernel
// The kernel for up to 64 rows where the two above and the tiles below are not faster (launch_lmhead).  Bound by streaming W
// from HBM once.  Kernel trace, average (fastest) of 60 launches that take three copies of W in turn, in us: V = 152064,
// d = 896, 32 rows 55.6 (53.6) for 292 MB, 5.2 TB/s, the kernels above 56.4; V = 32000, d = 768, 4 rows 10.2 (8.1), the kernels
// above 10.4; V = 50261, d = 1160, 15 rows 28.8 (27.6), with 64 x 64 tiles through LDS 39.2.
//   * Eight waves per workgroup.  KS of them share a 32-entry vocabulary tile, each taking its share of the k-blocks of 64; a
//     workgroup owns 8 / KS tiles and walks over the vocabulary.
//   * A wave reads its k-block of W as whole 128-byte lines, 8 lanes a row, PF k-blocks ahead of the one being multiplied,
//     and turns it through a wave-private LDS patch.  (Read straight into operand layout, where 16 consecutive lanes hold
//     16 different rows, a load instruction looks up 64 lines instead of 8 and W comes in at a quarter of the rate.)
//   * 16 * MT rows of H sit in LDS (rows padded by 16 bytes against bank conflicts), all of K at once where that fits, else
//     in chunks of kc columns: the next chunk is requested into registers at the start of a chunk's k-blocks.
//   * W is the row operand, so that an accumulator is [vocabulary][row].  The KS partial results meet in the patches, 32 rows
//     at a time, from where eight lanes add them, reduce the tile's softmax partials and store one whole 128-byte line of a
//     logits row past L2.
// Loads are never predicated (their number in flight has to be known): rows, vocabulary entries and k-blocks past the end
// re-read the last one.
constexpr int kStreamThreads = 512;
constexpr int kStreamHPieces(int MT) { return MT == 1 ? 8 : MT == 2 ? 8 : 12; }        // 16-byte pieces of an H chunk per thread
constexpr int kStreamMaxKC(int MT) { return kStreamHPieces(MT) * kStreamThreads * 8 / (MT * 16); }

template <int MT, int KS, int PF, bool CH>
__global__ __launch_bounds__(kStreamThreads) void k_lmhead_stream(int M, int d, int V, int n, int NT, int groups, int kc,
                                                                  int nchunks, int unit, int unit_inv, const uint16_t* __restrict__ W,
                                                                  const uint16_t* __restrict__ H, const float* __restrict__ temperature,
                                                                  float* __restrict__ L, float* __restrict__ pm, float* __restrict__ ps) {
    constexpr int kTiles = 8 / KS, VW = kTiles * 32;                        // vocabulary entries of a workgroup
    constexpr int SR = (MT == 1) ? 16 : 32;                                 // rows that meet in LDS at a time
    constexpr int HP = kStreamHPieces(MT), RP = (MT == 1) ? 16 : 32, CPP = kStreamThreads / (RP * 16);
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ float s_invt[MT * 16];
    const int hrow = kc * 2 + 16;
    unsigned char* const s_h = lds;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = wave % KS, tile = wave / KS, r16 = lane & 15, c = lane >> 4, lrow = lane >> 3, lchunk = lane & 7;
    unsigned char* const patches = lds + MT * 16 * hrow;                    // one per wave: 32 rows of 144 bytes
    unsigned char* const patch = patches + wave * kPatchBytes;
    const float my_temp = temperature[sequence_of(min(tid, M - 1), n)];     // used after the requests below

    // ---- H chunks: 16 lanes read 256 contiguous bytes of a row
    u32x4 hreg[HP];
    const char* const hbase = reinterpret_cast<const char*>(H);
    const int hr = (tid >> 4) % RP, hcg = (tid >> 4) / RP, hc = tid & 15;
    const int hcols = kc / (128 * CPP) + ((kc / 128) % CPP != 0);           // column passes of a chunk
    auto request_h = [&](int chunk) {
        int rp = RP;
        asm volatile("" : "+s"(rp));
#pragma unroll
        for (int q = 0; q < HP; ++q) {
            const int row = hr + (q % (MT * 16 / RP)) * rp, col = ((q / (MT * 16 / RP)) * CPP + hcg) * 128 + hc * 8;
            if (q / (MT * 16 / RP) < hcols) {
                const uint32_t k = min((uint32_t)(chunk * kc + col) * 2u, (uint32_t)d * 2u - 16u);
                hreg[q] = *reinterpret_cast<const u32x4*>(hbase + ((uint32_t)min(row, M - 1) * (uint32_t)d * 2u + k));
            }
        }
    };
    auto write_h = [&](int chunk) {
        int rp = RP;
        asm volatile("" : "+s"(rp));
#pragma unroll
        for (int q = 0; q < HP; ++q) {
            const int row = hr + (q % (MT * 16 / RP)) * rp, col = ((q / (MT * 16 / RP)) * CPP + hcg) * 128 + hc * 8;
            if (col < kc) {
                const u32x4 zero = {0u, 0u, 0u, 0u};
                *reinterpret_cast<u32x4*>(s_h + row * hrow + col * 2) = (chunk * kc + col < d) ? hreg[q] : zero;
            }
        }
    };

    // ---- W: step j of a chunk is k-block (chunk * kc / 64) + j * KS + ks of this wave's tile
    const int KB = (d + 63) / 64, kbc = kc / 64, steps = kbc / KS, psteps = (steps + PF - 1) / PF * PF;
    u32x4 ring[PF][4];                                                      // [slot][rows 8 i .. 8 i + 7], 8 lanes a row
    const char* wbase;
    uint32_t woff[4];
    auto aim = [&](int g) {
        const int v0 = g * VW + tile * 32;
        const int first = min(v0, V - 1);
        wbase = reinterpret_cast<const char*>(W) + (size_t)first * d * 2;
#pragma unroll
        for (int i = 0; i < 4; ++i) woff[i] = (uint32_t)min(8 * i + lrow, V - 1 - first) * (uint32_t)d * 2u;
    };
    // k-block (of a chunk) of this wave's step j: all of them, runs of `unit` in turn between two waves, or every fourth
    auto step_kb = [&](int j) {
        const int run = (KS == 2) ? (j * unit_inv) >> 16 : 0;
        return KS == 1 ? j : KS == 2 ? run * unit + ks * unit + j : j * KS + ks;
    };
    auto request_w = [&](int slot, int chunk, int j) {
        const int kb = min(chunk * kbc + step_kb(min(j, steps - 1)), KB - 1);
        const uint32_t k = min((uint32_t)(kb * 128 + lchunk * 16), (uint32_t)d * 2u - 16u);
#pragma unroll
        for (int i = 0; i < 4; ++i) ring[slot][i] = *reinterpret_cast<const u32x4*>(wbase + (woff[i] + k));
    };
    request_h(0);
    __builtin_amdgcn_sched_barrier(0);
    aim(blockIdx.x);
#pragma unroll
    for (int q = 0; q < PF; ++q) request_w(q, 0, q);
    __builtin_amdgcn_sched_barrier(0);
    write_h(0);
    if (tid < M) s_invt[tid] = inv_temperature(my_temp);
    lds_barrier();

    const bool ragged = (d & 63) != 0;
    for (int g = blockIdx.x;; g += gridDim.x) {
        const bool more = g + (int)gridDim.x < groups;
        f32x4 acc[2][MT];
#pragma unroll
        for (int vb = 0; vb < 2; ++vb)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[vb][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int chunk = 0; chunk < (CH ? nchunks : 1); ++chunk) {
            const bool last = !CH || chunk + 1 == nchunks;
            const bool restage = CH && (!last || more);
            if (restage) request_h(last ? 0 : chunk + 1);
            __builtin_amdgcn_sched_barrier(0);
            // PF steps; the slots they free are filled with the steps PF later (ahead = 0: of this chunk, 1: of the next
            // chunk or vocabulary group, 2: nothing is left to request)
            auto block = [&](int j0, auto ahead) {
#pragma unroll
                for (int q = 0; q < PF; ++q) {
                    const int j = j0 + q, kbl = step_kb(j);
                    const bool use = j < steps && chunk * kbc + kbl < KB;   // uniform
                    if (use) {                                              // LDS operations of one wave execute in order: no barrier
                        const bool out = ragged && (chunk * kbc + kbl) * 64 + lchunk * 8 >= d;
                        const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            *reinterpret_cast<u32x4*>(patch + (8 * i + lrow) * 144 + lchunk * 16) = out ? zero : ring[q][i];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (ahead.value == 0) request_w(q, chunk, j + PF);
                    if constexpr (ahead.value == 1) request_w(q, last ? 0 : chunk + 1, q);
                    __builtin_amdgcn_sched_barrier(0);
                    if (use) {
                        // operands of the next GM rows of 16 are read while the present ones are multiplied
                        constexpr int GM = MT < 4 ? MT : 4, NG = 2 * MT / GM;
                        int hr16 = 16 * hrow;
                        asm volatile("" : "+s"(hr16));                      // not worth a register per row block: recomputed
                        const unsigned char* const hp = s_h + r16 * hrow + kbl * 128 + c * 16;
                        bf16x8 w[2][2], hv[2][GM];
#pragma unroll
                        for (int p = 0; p < 2; ++p)
#pragma unroll
                            for (int vb = 0; vb < 2; ++vb) w[p][vb] = *reinterpret_cast<const bf16x8*>(patch + (vb * 16 + r16) * 144 + p * 64 + c * 16);
                        auto read_h = [&](int gi) {
                            const int p = gi / (MT / GM), t0 = gi % (MT / GM) * GM;
#pragma unroll
                            for (int i = 0; i < GM; ++i) hv[gi & 1][i] = *reinterpret_cast<const bf16x8*>(hp + (t0 + i) * hr16 + p * 64);
                        };
                        read_h(0);
#pragma unroll
                        for (int gi = 0; gi < NG; ++gi) {
                            if (gi + 1 < NG) read_h(gi + 1);
                            __builtin_amdgcn_sched_barrier(0);
                            const int p = gi / (MT / GM), t0 = gi % (MT / GM) * GM;
#pragma unroll
                            for (int i = 0; i < GM; ++i)
#pragma unroll
                                for (int vb = 0; vb < 2; ++vb)
                                    acc[vb][t0 + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[p][vb], hv[gi & 1][i], acc[vb][t0 + i], 0, 0, 0);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
            };
            for (int j0 = 0; j0 + PF < psteps; j0 += PF) block(j0, std::integral_constant<int, 0>{});
            if (last && !more) {
                block(psteps - PF, std::integral_constant<int, 2>{});
            } else {
                if (last) aim(g + gridDim.x);
                block(psteps - PF, std::integral_constant<int, 1>{});
            }
            if (restage) {
                lds_barrier();                                              // every wave is done with this chunk of H
                write_h(last ? 0 : chunk + 1);
                lds_barrier();
            }
        }

        // ---- the KS partial results meet, SR rows at a time
        int Vrow = V, NTrow = NT;
        asm volatile("" : "+s"(Vrow), "+s"(NTrow));                         // (addresses are not kept in registers across the loop above)
#pragma unroll
        for (int r0 = 0; r0 < MT * 16; r0 += SR) {
            if (r0 < M) {                                                   // uniform
#pragma unroll
                for (int i = 0; i < SR / 16; ++i)
#pragma unroll
                    for (int vb = 0; vb < 2; ++vb)
                        *reinterpret_cast<f32x4*>(patch + (i * 16 + r16) * 144 + vb * 64 + c * 16) = acc[vb][r0 / 16 + i];
                lds_barrier();
#pragma unroll
                for (int e = 0; e < SR * VW / 4; e += kStreamThreads) {
                    const int idx = e + tid, row = idx / (VW / 4), q4 = idx % (VW / 4);
                    if (SR * VW / 4 >= kStreamThreads || idx < SR * VW / 4) {
                        const unsigned char* part = patches + (q4 >> 3) * KS * kPatchBytes + row * 144 + (q4 & 7) * 16;
                        f32x4 x = *reinterpret_cast<const f32x4*>(part);
#pragma unroll
                        for (int w = 1; w < KS; ++w) x += *reinterpret_cast<const f32x4*>(part + w * kPatchBytes);
                        const int m = r0 + row, v = g * VW + 4 * q4;
                        const bool live = m < M;
                        const float it = live ? s_invt[m] : 1.f;
                        float sc[4], mx = -INFINITY;
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            sc[u] = (v + u < V) ? x[u] * it : -INFINITY;
                            mx = fmaxf(mx, sc[u]);
                        }
                        mx = fmaxf(mx, dpp_f32<kDppXor1>(mx));
                        mx = fmaxf(mx, dpp_f32<kDppXor2>(mx));
                        mx = fmaxf(mx, dpp_f32<kDppHalfMirror>(mx));
                        float sum = 0.f;
#pragma unroll
                        for (int u = 0; u < 4; ++u) sum += (sc[u] > -INFINITY) ? __expf(fmaf(x[u], it, -mx)) : 0.f;
                        sum += dpp_f32<kDppXor1>(sum);
                        sum += dpp_f32<kDppXor2>(sum);
                        sum += dpp_f32<kDppHalfMirror>(sum);
                        if (live && v < V) {
                            if ((q4 & 7) == 0) {
                                pm[(size_t)m * NTrow + v / kTileV] = mx;
                                ps[(size_t)m * NTrow + v / kTileV] = sum;
                            }
                            float* out = L + (size_t)m * Vrow + v;
                            if (v + 4 <= V) {
                                __builtin_nontemporal_store(f32x4u(x), reinterpret_cast<f32x4u*>(out));
                            } else {
#pragma unroll
                                for (int u = 0; u < 4; ++u)
                                    if (v + u < V) out[u] = x[u];
                            }
                        }
                    }
                }
                lds_barrier();                                              // the patches may be written again
            }
        }
        if (!more) break;
    }
}

// ---------------------------------------------------------------- bf16, many rows (more than 64, other hidden sizes from 33): tiled GEMM
// Workgroup tile BM (rows) x BN (vocabulary) x 64 (k), 8 waves, each a BM/2 x BN/4 block of 32x32 MFMA tiles (W as the row
// operand, so that the accumulator is [vocabulary][row] and the transposed epilogue applies).  Both operands are staged
// through LDS in two buffers; the operand fragments of k-step s+1 are read from LDS while the MFMAs of k-step s run, and the
// global loads of the next PF k-blocks are in flight in PF register sets -- one barrier per k-block.  A k-block of 64 is one
// whole 128-byte line of every row.  Rows padded by 16 bytes against bank conflicts.  Workgroups are numbered so that the row
// blocks that share a vocabulary block run back to back on the same XCD (workgroup w goes to XCD w % 8): W is then read from
// HBM once and from L2 afterwards.  Bound by how fast a workgroup takes in its operands and, with few k-blocks, by the logits'
// stores, which the larger tiles do not overlap with another tile's products.  Kernel trace, average (fastest) of 60 launches:
// 512 rows of V = 128256, d = 2048 339 us (314) = 0.79 PFLOP/s; 128 rows of V = 32000, d = 768 16.2 us (15.4), 30.1 when every tile
// was 256 x 256.
constexpr int kLBK = 64, kLRow = (kLBK + 8) * 2;                            // k-block; LDS row stride in bytes (144)
constexpr int kLCh = kLBK / 8;                                              // 16-byte chunks per row of a k-block
constexpr int kLargeThreads = 512;

// Off: type of a byte offset inside a tile (32 bits while a tile's rows span less than 4 GiB).
// NA: partial sums of a logit, over the k-blocks in turn, added in order at the end: those of the W-streaming kernel, whose
// waves share a tile in the same way (launch_stream).
template <int BM, int BN, int PF, typename Off, int NA = 1, bool PAST = true>
__global__ __launch_bounds__(kLargeThreads, (BM * BN <= 128 * 128 && NA <= 2) ? 4 : 2) void k_lmhead_tile(int M, int d, int V, int n, int NT,
                                                                int mblocks, const uint16_t* __restrict__ W,
                                                                const uint16_t* __restrict__ H,
                                                                const float* __restrict__ temperature,
                                                                float* __restrict__ L, float* __restrict__ pm,
                                                                float* __restrict__ ps) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ float s_invt[BM];
    constexpr int kStage = (BM + BN) * kLRow;
    constexpr int WP = BN * kLCh / kLargeThreads, HP = BM * kLCh / kLargeThreads;   // 16-byte pieces per thread
    constexpr int TV = BN / 128, TM = BM / 64;                                      // 32-wide tiles of a wave
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nn = lane & 31, half = lane >> 5;
    // XCD-aware numbering: workgroup w runs on XCD w % 8; consecutive slots of one XCD walk the row blocks
    // of one vocabulary block before moving to the next vocabulary block.
    const int w = blockIdx.x, xcd = w & 7, slot = w >> 3;
    const int mb = slot % mblocks, nb = (slot / mblocks) * 8 + xcd;
    const int m0 = mb * BM, v0 = nb * BN;
    if (v0 >= V) return;                                  // uniform: padding workgroups of the last XCD round
    const int wm = wave >> 2, wn = wave & 3;              // wave block: rows m0 + BM/2 * wm .., vocabulary v0 + BN/4 * wn ..
    const float my_temp = temperature[min(m0 + (tid & (BM - 1)), M - 1) / n];       // used after the requests below

    // ---- global -> register staging: piece q of a k-block is row q / 8, 16-byte chunk q % 8 (eight lanes a row).  Rows past
    //      the end re-read the last one (masked in the epilogue); chunks past the end of a row are zeroed.
    u32x4 rw[PF][WP], rh[PF][HP];
    const char* const wbase = reinterpret_cast<const char*>(W) + (size_t)v0 * d * 2;
    const char* const hbase = reinterpret_cast<const char*>(H) + (size_t)m0 * d * 2;
    Off wo[WP], ho[HP];
#pragma unroll
    for (int t = 0; t < WP; ++t) wo[t] = (Off)min((tid + t * kLargeThreads) / kLCh, V - 1 - v0) * (Off)d * 2u;
#pragma unroll
    for (int t = 0; t < HP; ++t) ho[t] = (Off)min((tid + t * kLargeThreads) / kLCh, M - 1 - m0) * (Off)d * 2u;
    const int KB = (d + kLBK - 1) / kLBK, ch = tid % kLCh;
    auto fetch = [&](int set, int kb) {                   // unconditional: the number of loads in flight has to be known
        const uint32_t k = min((uint32_t)min(kb, KB - 1) * 128u + (uint32_t)ch * 16u, (uint32_t)d * 2u - 16u);
#pragma unroll
        for (int t = 0; t < WP; ++t) rw[set][t] = *reinterpret_cast<const u32x4*>(wbase + (wo[t] + k));
#pragma unroll
        for (int t = 0; t < HP; ++t) rh[set][t] = *reinterpret_cast<const u32x4*>(hbase + (ho[t] + k));
    };
    auto stash = [&](int set, int kb) {
        unsigned char* sW = lds + (kb & 1) * kStage + tid / kLCh * kLRow + ch * 16;
        const bool out = kb * kLBK + ch * 8 >= d;
        const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < WP; ++t) *reinterpret_cast<u32x4*>(sW + t * (kLargeThreads / kLCh) * kLRow) = out ? zero : rw[set][t];
#pragma unroll
        for (int t = 0; t < HP; ++t) *reinterpret_cast<u32x4*>(sW + (BN + t * (kLargeThreads / kLCh)) * kLRow) = out ? zero : rh[set][t];
    };

    f32x16 acc[NA][TV][TM];                               // [partial sum][vocabulary tile][row tile]
#pragma unroll
    for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int a = 0; a < TV; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][a][b][r] = 0.f;

    auto multiply = [&](int kb, int i) {                  // i = kb % NA, known at compile time
        const unsigned char* sW = lds + (kb & 1) * kStage + (wn * 32 * TV + nn) * kLRow + half * 16;
        const unsigned char* sH = lds + (kb & 1) * kStage + (BN + wm * (BM / 2) + nn) * kLRow + half * 16;
        // operand fragments of k-step ks+1 are read from LDS while the MFMAs of k-step ks run
        bf16x8 wf[2][TV], hf[2][TM];
        auto read_frags = [&](int ks, int set) {
#pragma unroll
            for (int a = 0; a < TV; ++a) wf[set][a] = *reinterpret_cast<const bf16x8*>(sW + a * 32 * kLRow + ks * 32);
#pragma unroll
            for (int b = 0; b < TM; ++b) hf[set][b] = *reinterpret_cast<const bf16x8*>(sH + b * 32 * kLRow + ks * 32);
        };
        read_frags(0, 0);
#pragma unroll
        for (int ks = 0; ks < kLBK / 16; ++ks) {
            if (ks + 1 < kLBK / 16) read_frags(ks + 1, (ks + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);            // keep the reads ahead of the MFMAs they overlap with
#pragma unroll
            for (int a = 0; a < TV; ++a)
#pragma unroll
                for (int b = 0; b < TM; ++b)
                    acc[i][a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ks & 1][a], hf[ks & 1][b], acc[i][a][b], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

#pragma unroll
    for (int q = 0; q < PF; ++q) fetch(q, q);
    __builtin_amdgcn_sched_barrier(0);
    stash(0, 0);
    if (tid < BM) s_invt[tid] = inv_temperature(my_temp);
    fetch(0, PF);
    lds_barrier();
    // register set q holds k-block kb + 1 with (kb + 1) % PF = q: it goes to LDS after k-block kb is multiplied and is
    // refilled with the k-block PF later, except in the last PF k-blocks
    auto block = [&](int kb0, auto refill, auto first) {
#pragma unroll
        for (int q = 0; q < PF; ++q) {
            const int kb = kb0 + q;
            if (kb < KB) {
                multiply(kb, (first.value + q) % NA);
                if (kb + 1 < KB) stash((q + 1) % PF, kb + 1);
                if constexpr (refill.value) fetch((q + 1) % PF, kb + 1 + PF);
                lds_barrier();
            }
        }
    };
    static_assert(PF % NA == 0 || NA == 2 * PF, "block() runs PF k-blocks");
    constexpr std::integral_constant<int, 0> zero{};
    constexpr std::integral_constant<int, (NA > PF) ? PF : 0> next{};
    int kb0 = 0;
    if constexpr (NA > PF) {
        for (; kb0 + 2 * PF < KB; kb0 += 2 * PF) {
            block(kb0, std::true_type{}, zero);
            block(kb0 + PF, std::true_type{}, next);
        }
        if (kb0 + PF < KB) {
            block(kb0, std::true_type{}, zero);
            block(kb0 + PF, std::false_type{}, next);
        } else {
            block(kb0, std::false_type{}, zero);
        }
    } else {
        for (; kb0 + PF < KB; kb0 += PF) block(kb0, std::true_type{}, zero);
        block(kb0, std::false_type{}, zero);
    }
#pragma unroll
    for (int i = 1; i < NA; ++i)
#pragma unroll
        for (int a = 0; a < TV; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b) acc[0][a][b] += acc[i][a][b];
    // ---- epilogue: every wave turns its 32x32 blocks through a private patch carved from buffer 0
    unsigned char* tpatch = lds + wave * kPatchBytes;
#pragma unroll
    for (int a = 0; a < TV; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b)
            store_tile_32x32_t<PAST>(acc[0][a][b], m0 + wm * (BM / 2) + b * 32, v0 + wn * 32 * TV + a * 32, M, V, NT, s_invt - m0, L, pm, ps, tpatch);
}

// ---------------------------------------------------------------- bf16, more than 64 rows, hidden size a multiple of 64: operands straight to LDS
// The tiled GEMM above for the hidden sizes whose rows are whole lines: the same workgroup tiles, waves and order of sums (and so
// the same bits), but the operands go from memory to LDS without registers in between (global_load_lds, 16 bytes a lane), in SW
// stages of a k-block of W and SH of H; a wave keeps its registers for operand fragments, and nothing waits to write LDS.
// 256 x 256 tiles have room for three stages of W, which comes from memory, and two of H, which comes from L2 (0.8 % less than two
// of each).  A stage has rows of 128 bytes without padding; row r keeps its 16-byte pieces in the order piece ^ (r % 8), which the lanes
// bring about by the address they load from.  (Reads of 16 rows then meet on 32 of 64 banks, half of the 212 k LDS cycles a compute
// unit; the order piece ^ (r / 2 % 8) has no conflicts and gains 0.3 % with 256 x 256 tiles, but 128 rows of V = 32000, d = 768 took 26.5 us
// with it instead of 24.7 back to back on W in the last-level cache, for a reason not found.)
// One barrier per k-block, before the products of its last k-step: by then its last fragments are in registers and the stage is
// free, and the next k-block's first fragments are read while those products run.  (With the barrier at the k-block's end its first
// fragments were waited for: 333 us a draft step, 323.  The last k-blocks are waited for one by one too: with everything on its way
// waited for at once, 128 rows of V = 32000, d = 768, four stages, took 26.0 us instead of 24.9; 26.3 with the barrier at the end.)  The loads are written in assembly (they have no destination
// register): with the builtin the compiler waits for all LDS reads in flight at every second step, 256 us instead of 232 for the
// product alone below.
// What bounds it, 512 rows of V = 128256, d = 2048 (269 GFLOP, a draft step 304 us, 327 before): the loop without loads 178 us, with
// them 230, with the epilogue and its 263 MB of logits, which all workgroups store at about the same times, 283, launches apart; 188, 265
// and 315 on average back to back.  The matrix cores are busy for 76, 60 and 47 % of the cycles, at 1.9 GHz: the clock follows the power.  Measured and not kept:
// k-blocks walked from a different one in every vocabulary block, so that workgroups read different channels (no change).
// (M0 is put back: the compiler does not let it be named as clobbered, and keeps what it has in it.)
__device__ __forceinline__ void dma_lines(const char* base, const uint32_t (&off)[4], uint32_t lds, uint32_t step) {
    uint32_t m0;
    // (the waits: M0 written before an LDS load, and a scalar that may have come from a vector instruction)
    asm volatile("s_mov_b32 %0, m0\n\ts_nop 4\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %7\n\ts_add_u32 m0, m0, %2\n\t"
                 "s_nop 0\n\tglobal_load_lds_dwordx4 %4, %7\n\ts_add_u32 m0, m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %5, %7\n\t"
                 "s_add_u32 m0, m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %6, %7\n\ts_mov_b32 m0, %0"
                 : "=&s"(m0) : "s"(lds), "s"(step), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base) : "memory", "scc");
}
__device__ __forceinline__ void dma_lines(const char* base, const uint32_t (&off)[2], uint32_t lds, uint32_t step) {
    uint32_t m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_nop 4\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %5\n\ts_add_u32 m0, m0, %2\n\t"
                 "s_nop 0\n\tglobal_load_lds_dwordx4 %4, %5\n\ts_mov_b32 m0, %0"
                 : "=&s"(m0) : "s"(lds), "s"(step), "v"(off[0]), "v"(off[1]), "s"(base) : "memory", "scc");
}

template <int BM, int BN, int SW, int SH, bool PAST>
__global__ __launch_bounds__(kLargeThreads, 2) void k_lmhead_dma(int M, int d, int V, int n, int NT, int mblocks, const uint16_t* __restrict__ W,
                                                                 const uint16_t* __restrict__ H, const float* __restrict__ temperature,
                                                                 float* __restrict__ L, float* __restrict__ pm, float* __restrict__ ps) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int kRow = kLBK * 2, kStW = BN * kRow, kStH = BM * kRow;       // SW stages of W, then SH of H
    constexpr int TV = BN / 128, TM = BM / 64;                              // 32-wide tiles of a wave
    constexpr int WI = BN / 64, HI = BM / 64;                               // loads of a wave per stage: 8 rows of 128 bytes each
    constexpr uint32_t kStep = 8 * 8 * kRow;                                // LDS bytes from one of a wave's loads to its next
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nn = lane & 31, half = lane >> 5;
    // (numbering as above: row blocks of a vocabulary block back to back on one XCD)
    const int w = blockIdx.x, xcd = w & 7, slot = w >> 3;
    const int mb = slot % mblocks, nb = (slot / mblocks) * 8 + xcd;
    const int m0 = mb * BM, v0 = nb * BN;
    if (v0 >= V) return;                                                    // uniform: padding workgroups of the last XCD round
    const int wm = wave >> 2, wn = wave & 3;
    const float my_temp = temperature[min(m0 + (tid & (BM - 1)), M - 1) / n];       // used after the loop
    const int KB = d / kLBK;
    const char* const wbase = reinterpret_cast<const char*>(W) + (size_t)v0 * d * 2;
    const char* const hbase = reinterpret_cast<const char*>(H) + (size_t)m0 * d * 2;
    uint32_t wo[WI], ho[HI];                                                // rows past the end re-read the last one (masked in the epilogue)
    {
        const int r = lane >> 3;
        const uint32_t piece = (uint32_t)((lane & 7) ^ r) * 16u;
#pragma unroll
        for (int i = 0; i < WI; ++i) wo[i] = (uint32_t)min((i * 8 + wave) * 8 + r, V - 1 - v0) * (uint32_t)d * 2u + piece;
#pragma unroll
        for (int i = 0; i < HI; ++i) ho[i] = (uint32_t)min((i * 8 + wave) * 8 + r, M - 1 - m0) * (uint32_t)d * 2u + piece;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds + (uint32_t)wave * 8u * kRow;
    auto request_w = [&](int kb, int stage) { dma_lines(wbase + kb * kRow, wo, lds0 + (uint32_t)(stage * kStW), kStep); };       // kb < KB
    auto request_h = [&](int kb, int stage) { dma_lines(hbase + kb * kRow, ho, lds0 + (uint32_t)(SW * kStW + stage * kStH), kStep); };

    f32x16 acc[TV][TM];                                                     // [vocabulary tile][row tile]
#pragma unroll
    for (int a = 0; a < TV; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    const uint32_t wrow = (uint32_t)(wn * 32 * TV + nn) * kRow, hrow = (uint32_t)(SW * kStW) + (uint32_t)(wm * (BM / 2) + nn) * kRow, turn = (uint32_t)(nn & 7);
    bf16x8 wf[2][TV], hf[2][TM];                                            // fragments of two k-steps of 16
    int stw = 0, sth = 0;                                                   // stages of the present k-block
    auto read_frags = [&](int ks, int set) {
        const unsigned char* sW = lds + stw * kStW + wrow;
        const unsigned char* sH = lds + sth * kStH + hrow;
        const uint32_t c = ((uint32_t)(2 * ks + half) ^ turn) * 16u;
#pragma unroll
        for (int a = 0; a < TV; ++a) wf[set][a] = *reinterpret_cast<const bf16x8*>(sW + a * 32 * kRow + c);
#pragma unroll
        for (int b = 0; b < TM; ++b) hf[set][b] = *reinterpret_cast<const bf16x8*>(sH + b * 32 * kRow + c);
    };
    auto products = [&](int set) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 0; a < TV; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[set][a], hf[set][b], acc[a][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };

    static_assert(SW == SH || SW == SH + 1, "the order of requests below");
#pragma unroll
    for (int q = 0; q < SW; ++q) {
        request_w(q, q);
        if (q < SH) request_h(q, q);
    }
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((SW - 1) * WI + (SH - 1) * HI) : "memory");
    read_frags(0, 0);
    auto step = [&](int kb, auto refill, auto left) {
#pragma unroll
        for (int ks = 0; ks < kLBK / 16 - 1; ++ks) {                        // fragments of k-step ks + 1 are read while ks is multiplied
            read_frags(ks + 1, (ks + 1) & 1);
            products(ks & 1);
        }
        // The stage's last fragments are in registers: it is free once all waves are here.  k-block kb + 1 is there once no more than what
        // a wave asked for after that (left) is outstanding.  Its first fragments are read while the last products run.
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(left.value) : "memory");
        if constexpr (refill.value) {
            request_h(kb + SH, sth);
            request_w(min(kb + SW, KB - 1), stw);
        }
        stw = (stw + 1 == SW) ? 0 : stw + 1;
        sth = (sth + 1 == SH) ? 0 : sth + 1;
        read_frags(0, 0);
        products(1);
    };
    static_assert(kLBK == 64, "the last of a stage's k-steps uses the second set");
    int kb = 0;
    for (; kb + SH < KB; ++kb) step(kb, std::true_type{}, std::integral_constant<int, (SW - 2) * WI + (SH - 2) * HI>{});
    auto tail = [&](auto t) {                                               // the last SH k-blocks (a third stage of W: what it was asked for again)
        constexpr int pairs = SH - 2 - t.value > 0 ? SH - 2 - t.value : 0;
        if constexpr (t.value < SH) step(kb + t.value, std::false_type{}, std::integral_constant<int, pairs * (WI + HI) + (SW - SH) * WI>{});
    };
    static_assert(SH <= 4, "tail");
    tail(std::integral_constant<int, 0>{});
    tail(std::integral_constant<int, 1>{});
    tail(std::integral_constant<int, 2>{});
    tail(std::integral_constant<int, 3>{});
    constexpr int kPT = BN / kTileV, kPS = BM * kPT;                        // partials of a row; of all rows
    float* const s_invt = reinterpret_cast<float*>(lds + 16 * kPatchBytes);
    float* const s_part = s_invt + BM;                                      // [2][BM][kPT]
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");             // nothing is on its way to LDS any more, nothing is read from it
    __syncthreads();
    if (tid < BM) s_invt[tid] = inv_temperature(my_temp);
    __syncthreads();
    // ---- epilogue: every wave turns its 32x32 blocks through private patches carved from the stages
    unsigned char* const tpatch = lds + wave * 2 * kPatchBytes;
    if (v0 + BN > V) {                                                      // uniform: the last vocabulary block
#pragma unroll
        for (int a = 0; a < TV; ++a)
#pragma unroll
            for (int b = 0; b < TM; ++b)
                store_tile_32x32_t<PAST>(acc[a][b], m0 + wm * (BM / 2) + b * 32, v0 + wn * 32 * TV + a * 32, M, V, NT, s_invt - m0, L, pm, ps, tpatch);
        return;
    }
    const int lr = wm * (BM / 2);
    store_full_tiles<PAST, TV, TM, kPT, kPS>(acc, M - m0 - lr, s_invt + lr, s_part + lr * kPT + wn * TV, L + (size_t)(m0 + lr) * V + v0 + wn * 32 * TV, V, tpatch);
    lds_barrier();
#pragma unroll
    for (int t = tid; t < 2 * BM * (kPT / 4); t += kLargeThreads) {
        const int q = t % (kPT / 4), row = t / (kPT / 4) % BM, arr = t / (kPT / 4) / BM;
        const f32x4 x = *reinterpret_cast<const f32x4*>(s_part + arr * kPS + row * kPT + 4 * q);
        if (m0 + row < M) *reinterpret_cast<f32x4u*>((arr == 0 ? pm : ps) + (size_t)(m0 + row) * NT + v0 / kTileV + 4 * q) = f32x4u(x);
    }
}

// ---------------------------------------------------------------- fp32 operands: one output per thread
// Workgroup = 8 rows x 32 vocabulary entries; a half-wave shares one row, so the tile partials are a
// half-wave reduction.  Only the tiny correctness configuration stores fp32 weights.
__global__ __launch_bounds__(kBlock) void k_lmhead_f32(int M, int d, int V, int n, int NT,
                                                       const float* __restrict__ W, const float* __restrict__ H,
                                                       const float* __restrict__ temperature,
                                                       float* __restrict__ L, float* __restrict__ pm,
                                                       float* __restrict__ ps) {
    const int tid = threadIdx.x;
    const int m = blockIdx.y * 8 + (tid >> 5);
    const int v = blockIdx.x * kTileV + (tid & 31);
    const bool live = (m < M);
    float s = -INFINITY;
    if (live && v < V) {
        const float* w = W + (size_t)v * d;
        const float* h = H + (size_t)m * d;
        double acc = 0.0;
        for (int k = 0; k < d; ++k) acc += (double)h[k] * (double)w[k];
        const float x = (float)acc;
        L[(size_t)m * V + v] = x;
        s = x * row_inv_temperature(temperature, m, n);
    }
    const float mx = half_max(s);
    const float e = (s > -INFINITY) ? __expf(s - mx) : 0.f;
    const float sum = half_sum(e);
    if (live && (tid & 31) == 0) {
        pm[(size_t)m * NT + blockIdx.x] = mx;
        ps[(size_t)m * NT + blockIdx.x] = sum;
    }
}

// k-blocks of 128 per chunk of the chunked kernel (hidden sizes that are at least two times 512, 768 or 896), 0 for other sizes.
// With two row blocks the 512-wide chunk is the one that keeps the H prefetch in registers without spills.
static int skinny_kc_kh(const tabed_cfg& c, int M) {
    const int two[3] = {4, 6, 7}, one[3] = {6, 4, 7};
    for (int KH : (M > 32 ? two : one))
        if (c.d % (KH * 128) == 0 && c.d / (KH * 128) >= 2) return KH;
    return 0;
}

template <int KH, int MT>
static hipError_t launch_skinny_kc_t(const ProfScope* prof, const tabed_cfg& c, const WsLayout& Lay, int M, const void* W,
                               const void* H, const float* temperature, float* logits, float* pm, float* ps,
                               hipStream_t s) {
    const size_t lds = (size_t)MT * 32 * (KH * 256 + 16) + (size_t)kSkinnyWaves * kPatchBytes;
    static std::once_flag attr_once;
    static hipError_t attr_rc = hipSuccess;
    if (raise_lds_limit(&k_lmhead_skinny_kc<KH, MT>, lds, attr_once, attr_rc) != hipSuccess) return attr_rc;
    const int num_tiles = Lay.NT, groups = (num_tiles + 3) / 4;
    const dim3 grid(groups < 256 ? groups : 256);
    launch(prof, k_lmhead_skinny_kc<KH, MT>, grid, dim3(kSkinnyThreads), lds, s, M, c.V, c.n, Lay.NT, num_tiles,
           c.d / (KH * 128), static_cast<const uint16_t*>(W), static_cast<const uint16_t*>(H), temperature, logits, pm, ps);
    return hipSuccess;
}

static hipError_t launch_skinny_kc(const ProfScope* prof, int KH, const tabed_cfg& c, const WsLayout& Lay, int M,
                             const void* W, const void* H, const float* temperature, float* logits, float* pm,
                             float* ps, hipStream_t s) {
#define TABED_SKINNY_KC(KH_)                                                                                         \
    if (KH == KH_)                                                                                                   \
        return M <= 32 ? launch_skinny_kc_t<KH_, 1>(prof, c, Lay, M, W, H, temperature, logits, pm, ps, s)           \
                       : launch_skinny_kc_t<KH_, 2>(prof, c, Lay, M, W, H, temperature, logits, pm, ps, s);
    TABED_SKINNY_KC(4) TABED_SKINNY_KC(6) TABED_SKINNY_KC(7)
#undef TABED_SKINNY_KC
    return hipErrorInvalidValue;
}

// (d = 1024 up to 32 rows: two blocks of 32 rows and the patches do not fit LDS)
static bool skinny_applies(const tabed_cfg& c, int M) {
    return c.d == 4 * 128 || c.d == 6 * 128 || c.d == 7 * 128 || (c.d == 8 * 128 && M <= 32);
}

// Up to 32 rows: whether the kernels with a compile-time hidden size run, or the W-streaming kernel.  Whole draft steps
// replayed back to back on one copy of W, in us, those / streaming:
//   d = 512: always (V = 32000, 32 rows 11.3 / 13.7; V = 65536, 8 rows 18.6 / 19.9), except for vocabularies that the streaming
//     kernel cuts finer (V = 8000: 0.9 of the time);
//   17 to 32 rows, d = 768 and 896: with few groups of 128 entries a workgroup (V = 20000, d = 896 12.3 / 13.6, V = 40000 3 % less;
//     V = 65536 equal);
//   17 to 32 rows, H in chunks or d = 1024: V = 40000, d = 2560 45.6 / 49.6; V = 20000, d = 3584 6 % less, d = 1024 13.4 / 14.5; but
//     rows that lie a multiple of 2 KB apart only while W fits the 256 MB of the last-level cache (d = 2048 V = 65536 3 % less,
//     V = 100000 9 % more; d = 4096 V = 32000 4 % less, V = 40000 7 % more).
static bool skinny_wins(const tabed_cfg& c, int M) {
    if (c.V <= 128 * 128) return false;
    if (c.d == 512) return true;
    if (M <= 16) return false;
    if (c.d % 1024 == 0) return (long)c.V * c.d <= 1l << 27;
    return c.V <= 384 * 128 || !skinny_applies(c, M);
}

template <int KH, int MT>
static hipError_t launch_skinny_t(const ProfScope* prof, const tabed_cfg& c, const WsLayout& Lay, int M, const void* W, const void* H,
                            const float* temperature, float* logits, float* pm, float* ps, hipStream_t s) {
    const size_t lds = (size_t)MT * 32 * (KH * 256 + 16) + (size_t)kSkinnyWaves * kPatchBytes;
    static std::once_flag attr_once;                   // raise the dynamic-LDS limit of this instantiation once
    static hipError_t attr_rc = hipSuccess;
    if (raise_lds_limit(&k_lmhead_skinny<KH, MT>, lds, attr_once, attr_rc) != hipSuccess) return attr_rc;
    const int num_tiles = Lay.NT;
    int cus = 256;
    const int groups = (num_tiles + 3) / 4;
    const dim3 grid(groups < cus ? groups : cus);
    launch(prof, k_lmhead_skinny<KH, MT>, grid, dim3(kSkinnyThreads), lds, s, M, c.V, c.n, Lay.NT, num_tiles,
                       static_cast<const uint16_t*>(W), static_cast<const uint16_t*>(H), temperature, logits, pm, ps);
    return hipSuccess;
}

static hipError_t launch_skinny(const ProfScope* prof, const tabed_cfg& c, const WsLayout& Lay, int M, const void* W, const void* H,
                          const float* temperature, float* logits, float* pm, float* ps, hipStream_t s) {
    const int KH = c.d / 128;
#define TABED_SKINNY(KH_)                                                                                         \
    if (KH == KH_)                                                                                                \
        return M <= 32 ? launch_skinny_t<KH_, 1>(prof, c, Lay, M, W, H, temperature, logits, pm, ps, s)           \
                       : launch_skinny_t<KH_, 2>(prof, c, Lay, M, W, H, temperature, logits, pm, ps, s);
    TABED_SKINNY(4) TABED_SKINNY(6) TABED_SKINNY(7)
#undef TABED_SKINNY
    if (KH == 8 && M <= 32) return launch_skinny_t<8, 1>(prof, c, Lay, M, W, H, temperature, logits, pm, ps, s);
    return hipErrorInvalidValue;
}

template <int MT, int KS, int PF, bool CH>
static hipError_t launch_stream_t(const ProfScope* prof, const tabed_cfg& c, const WsLayout& Lay, int kc, int nchunks, int unit,
                                  const void* W, const void* H, const float* temperature, float* logits, float* pm, float* ps,
                                  hipStream_t s) {
    constexpr int VW = 8 / KS * 32;
    const size_t lds = (size_t)MT * 16 * (kc * 2 + 16) + 8 * (size_t)kPatchBytes;
    static std::once_flag once;
    static hipError_t rc = hipSuccess;
    if (raise_lds_limit(&k_lmhead_stream<MT, KS, PF, CH>, (size_t)MT * 16 * (kStreamMaxKC(MT) * 2 + 16) + 8 * (size_t)kPatchBytes, once, rc) != hipSuccess) return rc;
    const int groups = (c.V + VW - 1) / VW;
    const int grid = std::min(groups, lds <= 80 * 1024 ? 512 : 256);       // persistent: two workgroups a compute unit where LDS allows
    launch(prof, k_lmhead_stream<MT, KS, PF, CH>, dim3(grid), dim3(kStreamThreads), lds, s, Lay.M, c.d, c.V, c.n, Lay.NT, groups, kc,
           nchunks, unit, 65536 / unit + 1, static_cast<const uint16_t*>(W), static_cast<const uint16_t*>(H), temperature, logits, pm, ps);
    return hipSuccess;
}

template <int MT, int KS>
static hipError_t launch_stream_k(const ProfScope* prof, const tabed_cfg& c, const WsLayout& Lay, int unit, const void* W, const void* H,
                                  const float* temperature, float* logits, float* pm, float* ps, hipStream_t s) {
    const int granule = std::max(128, 64 * KS * unit), most = kStreamMaxKC(MT) / granule * granule;
    const int nchunks = (c.d + most - 1) / most;
    const int kc = (((c.d + nchunks - 1) / nchunks) + granule - 1) / granule * granule, steps = kc / 64 / KS;
    // three or four k-blocks ahead: whichever divides a chunk's steps with less of a remainder
    const bool four = KS <= 2 && (steps + 3) / 4 * 4 <= (steps + 2) / 3 * 3;
#define TABED_STREAM(PF_, CH_) return launch_stream_t<MT, KS, PF_, CH_>(prof, c, Lay, kc, nchunks, unit, W, H, temperature, logits, pm, ps, s)
    if constexpr (KS <= 2)
        if (four) { if (nchunks > 1) TABED_STREAM(4, true); else TABED_STREAM(4, false); }
    if (nchunks > 1) TABED_STREAM(3, true); else TABED_STREAM(3, false);
#undef TABED_STREAM
}

// Waves per vocabulary tile, and which k-blocks each of them adds up.  A logit's last bit depends on this order, and with 1e5
// bins a sampled token on the last bits of all of them.  The order is a function of row count (up to 64, more; for
// the first line's sizes also up to 32, 33 to 64), hidden size and vocabulary, and nothing else.  (Times: back to back on one
// copy of W; a copy that is not cached adds 1 to 2 us.)
//   * d = 512, 768, 896 and multiples, up to 64 rows: two waves, runs of half a chunk in turn.  The chunk is 768, 512 or 896 wide
//     up to 32 rows (the first that divides d; d = 1024 is one chunk), 512, 768 or 896 wide from 33 rows on; the streaming
//     kernel and the two above share an order, so that which of them runs does not matter.
//   * other hidden sizes, up to 64 rows: one wave, all k-blocks in order, where groups of 128 entries would not be one round of a
//     group per compute unit (V = 38000, d = 1280, 4 rows: 18.9 us, 22.1 with two waves).  Up to there two waves take turns
//     (V = 32000, d = 1280, 20 rows: 15.0 us, 17.1 with one).
//   * vocabularies of at most 128 groups: four waves a tile (V = 10000, d = 1160, 20 rows: 9.0 us, 11.0 with two, 17.9 with one),
//     k-blocks in turn; from 33 rows on not for the first line's sizes.  (The tiles that take 33 to 64 rows keep as many partial sums, NA.  One sum over all k-blocks there had 1.4
//     to 1.8 times the error: V = 8000, d = 640, 48 rows 14.2e-8 relative, 8.0e-8 with four; V = 32000, d = 1160 19.8e-8, 13.7e-8
//     with two.)
//   * more than 64 rows: all k-blocks in order.
template <int MT>
static hipError_t launch_stream(const ProfScope* prof, const tabed_cfg& c, const WsLayout& Lay, const void* W, const void* H,
                                const float* temperature, float* logits, float* pm, float* ps, hipStream_t s) {
    int run = (c.d == 1024) ? 8 : 0;
    for (int KH : {6, 4, 7}) if (run == 0 && c.d % (KH * 128) == 0) run = KH;
    if (c.V <= 128 * 128) return launch_stream_k<MT, 4>(prof, c, Lay, 1, W, H, temperature, logits, pm, ps, s);
    if (run == 0 && c.V > 256 * 128) return launch_stream_k<MT, 1>(prof, c, Lay, 1, W, H, temperature, logits, pm, ps, s);
    return launch_stream_k<MT, 2>(prof, c, Lay, run ? run : 1, W, H, temperature, logits, pm, ps, s);
}

template <int BM, int BN, int PF, typename Off, int NA = 1, bool PAST = true>
static hipError_t launch_tile(const ProfScope* prof, const tabed_cfg& c, const WsLayout& Lay, int M, const void* W, const void* H,
                              const float* temperature, float* logits, float* pm, float* ps, hipStream_t s) {
    const size_t lds = 2 * (size_t)(BM + BN) * kLRow;
    static std::once_flag once;
    static hipError_t rc = hipSuccess;
    if (raise_lds_limit(&k_lmhead_tile<BM, BN, PF, Off, NA, PAST>, lds, once, rc) != hipSuccess) return rc;
    const int mblocks = (M + BM - 1) / BM, nblocks = (c.V + BN - 1) / BN;
    const int nrounds = (nblocks + 7) / 8;             // vocabulary blocks are dealt to the 8 XCDs in rounds
    launch(prof, k_lmhead_tile<BM, BN, PF, Off, NA, PAST>, dim3(nrounds * mblocks * 8), dim3(kLargeThreads), lds, s, M, c.d, c.V, c.n, Lay.NT, mblocks,
           static_cast<const uint16_t*>(W), static_cast<const uint16_t*>(H), temperature, logits, pm, ps);
    return hipSuccess;
}

template <int BM, int BN, int SW, int SH, bool PAST>
static hipError_t launch_dma(const ProfScope* prof, const tabed_cfg& c, const WsLayout& Lay, int M, const void* W, const void* H,
                             const float* temperature, float* logits, float* pm, float* ps, hipStream_t s) {
    constexpr size_t lds = std::max((size_t)(SW * BN + SH * BM) * kLBK * 2, (size_t)16 * kPatchBytes + BM * 4 + 2 * BM * (BN / kTileV) * 4);
    static std::once_flag once;
    static hipError_t rc = hipSuccess;
    if (raise_lds_limit(&k_lmhead_dma<BM, BN, SW, SH, PAST>, lds, once, rc) != hipSuccess) return rc;
    const int mblocks = (M + BM - 1) / BM, nblocks = (c.V + BN - 1) / BN;
    const int nrounds = (nblocks + 7) / 8;             // vocabulary blocks are dealt to the 8 XCDs in rounds
    launch(prof, k_lmhead_dma<BM, BN, SW, SH, PAST>, dim3(nrounds * mblocks * 8), dim3(kLargeThreads), lds, s, M, c.d, c.V, c.n, Lay.NT, mblocks,
           static_cast<const uint16_t*>(W), static_cast<const uint16_t*>(H), temperature, logits, pm, ps);
    return hipSuccess;
}

hipError_t launch_lmhead(const tabed_cfg& c, const WsLayout& Lay, char* ws, const void* W, const void* H,
                         const float* temperature, float* logits, hipStream_t s, int prof_id) {
    ProfScope prof(prof_id, s);
    float* pm = reinterpret_cast<float*>(ws + Lay.off_pm);
    float* ps = reinterpret_cast<float*>(ws + Lay.off_ps);
    const int M = Lay.M;
    hipError_t e = hipSuccess;
    if (c.w_dtype == 0) {
        const dim3 grid(Lay.NT, (M + 7) / 8);
        launch(&prof, k_lmhead_f32, grid, dim3(kBlock), 0, s, M, c.d, c.V, c.n, Lay.NT,
                           static_cast<const float*>(W), static_cast<const float*>(H), temperature, logits, pm, ps);
    } else if (c.d > (1 << 22)) {                       // rows of more than 8 MB: 64-bit offsets inside a tile
        e = launch_tile<128, 128, 2, uint64_t>(&prof, c, Lay, M, W, H, temperature, logits, pm, ps, s);
    } else if (M <= 64 && skinny_applies(c, M) && (M > 32 || skinny_wins(c, M))) {
        e = launch_skinny(&prof, c, Lay, M, W, H, temperature, logits, pm, ps, s);
    } else if (M <= 64 && skinny_kc_kh(c, M) != 0 && (M > 32 || skinny_wins(c, M))) {
        e = launch_skinny_kc(&prof, skinny_kc_kh(c, M), c, Lay, M, W, H, temperature, logits, pm, ps, s);
    } else if (M <= 16) {
        e = launch_stream<1>(&prof, c, Lay, W, H, temperature, logits, pm, ps, s);
    } else if (M <= 32) {
        e = launch_stream<2>(&prof, c, Lay, W, H, temperature, logits, pm, ps, s);
    } else if (M <= 64 && c.V <= 128 * 128 && c.d > 512) {
        e = launch_stream_k<4, 4>(&prof, c, Lay, 1, W, H, temperature, logits, pm, ps, s);
    } else if (M <= 64) {
        // 64 rows in one tile.  Whole draft steps in us: V = 32000, 64 rows, d = 1000 19.3, with W streamed (H in two chunks) 30.1;
        // d = 64 10.4 / 11.4; V = 16384, 48 rows, d = 320 10.5 / 10.9; d = 640 the other way round, 12.2 / 11.9, and V = 8000, d = 1920
        // 4 % less streamed with four waves a tile.  The partial sums cost 0.1 to 0.3 us.
        if (c.V <= 128 * 128) e = launch_tile<64, 128, 2, uint32_t, 4>(&prof, c, Lay, M, W, H, temperature, logits, pm, ps, s);
        else if (c.V <= 256 * 128) e = launch_tile<64, 128, 2, uint32_t, 2>(&prof, c, Lay, M, W, H, temperature, logits, pm, ps, s);
        else e = launch_tile<64, 128, 2, uint32_t>(&prof, c, Lay, M, W, H, temperature, logits, pm, ps, s);
    } else {
        // the largest tile that still gives the chip three workgroups for every four compute units (a tile reads
        // (BM + BN) / (BM BN) operand elements per product): fastest launches of 312 / 340 / 371 us for 256 x 256, 128 x 256,
        // 128 x 128 at 512 rows of V = 128256, d = 2048; 89 / 103 / 102 at 256 rows of V = 100000, d = 1024; but 30 / 18.1 / 14.4 at
        // 128 rows of V = 32000, d = 768, where they are 125, 125 and 250 workgroups; and the largest one too where the next would
        // take a second round over the compute units: a draft step of 256 rows of V = 40000, d = 1024 48 us with 157 workgroups of
        // 256 x 256, 54 with 314
        auto tiles = [&](int bm, int bn) { return (long)((M + bm - 1) / bm) * ((c.V + bn - 1) / bn); };
        // Rows of whole lines: operands go straight to LDS.  Whole draft steps in us, straight / through registers: 337 / 354 at 512
        // rows of V = 128256, d = 2048; 66.1 / 70.5 at 160 rows of 50261, 1152; 24.9 / 25.4 at 128 of 32000, 768; 87.5 / 94.3 at 96 of
        // 152064, 896; 76.4 / 76.3 at 96 of 32000, 4096; 19.7 / 19.8 at 256 of 9000, 512.  With one or two k-blocks there is nothing to have in
        // flight: 16.3 / 15.9 at 400 rows of 8000, 64, 33.6 / 33.1 at 256 of 65536, 128.
        const bool past = past_l2(c.V, c.d, M);
#define TABED_ROWS(FN_, ...)                                                               \
    past ? FN_<__VA_ARGS__, true>(&prof, c, Lay, M, W, H, temperature, logits, pm, ps, s)    \
         : FN_<__VA_ARGS__, false>(&prof, c, Lay, M, W, H, temperature, logits, pm, ps, s)
        const bool lines = c.d % kLBK == 0 && c.d >= 512;
        if (lines && M > 128 && (tiles(256, 256) >= 192 || tiles(128, 256) > 256))
            e = TABED_ROWS(launch_dma, 256, 256, 3, 2);
        else if (lines && tiles(128, 256) >= 192)
            e = TABED_ROWS(launch_dma, 128, 256, 3, 3);
        else if (lines && tiles(128, 128) > 256)       // two workgroups a compute unit (192 rows of 20000, 896 33.7 us with one, 29.0; 30.2 through registers)
            e = TABED_ROWS(launch_dma, 128, 128, 2, 2);
        else if (lines)                                // (at most 256 tiles: M V reaches 2^22 with whole ones only, and such a V goes past L2)
            e = launch_dma<128, 128, 4, 4, true>(&prof, c, Lay, M, W, H, temperature, logits, pm, ps, s);
        else if (M > 128 && (tiles(256, 256) >= 192 || tiles(128, 256) > 256))
            e = TABED_ROWS(launch_tile, 256, 256, 1, uint32_t, 1);
        else if (tiles(128, 256) >= 192) e = TABED_ROWS(launch_tile, 128, 256, 2, uint32_t, 1);
        else e = TABED_ROWS(launch_tile, 128, 128, 2, uint32_t, 1);
#undef TABED_ROWS
    }
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

}  // namespace tabed
