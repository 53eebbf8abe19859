// Vocabulary-wide passes of a TABED round on gfx950: ensemble + draft token (Alg. 1 (W-Avg and Sample steps)),
// target statistics + per-draft KL + accept chain (Sec. 3 items 2-3, Sec. 5.1), corrected / bonus token
// (Sec. 3 item 3), window + weights (Alg. 1 (weight-selection step), App. B.2).  All of them are HBM- or latency-bound:
// DPP lane exchanges and a few LDS words do the reductions, fp64 carries the cross-wave and cross-workgroup
// sums, and partial results cross workgroups through device-scope atomic stores that are waited for before an
// arrival counter moves (no cache-flushing fences).
#include <type_traits>

#include "device_utils.h"
#include "internal.h"

namespace tabed {

// =====================================================================================================
// Small kernels: workspace init, Philox dump, weights.
// =====================================================================================================
__global__ void k_fill_u32(uint32_t* p, int count) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0u;
}

hipError_t launch_ws_init(const tabed_cfg& c, const WsLayout& L, char* ws, hipStream_t s) {
    const int count = 5 * c.B * L.TS;
    launch(nullptr, k_fill_u32, dim3((count + 255) / 256), dim3(256), 0, s,
                       reinterpret_cast<uint32_t*>(ws + L.off_tickets), count);
    return hipGetLastError();
}

__global__ void k_null() {}

hipError_t launch_null(hipStream_t s) {
    ProfScope prof(TABED_K_NULL, s);
    launch(&prof, k_null, dim3(1), dim3(64), 0, s);
    return hipGetLastError();
}

__global__ void k_philox(uint64_t seed, uint64_t round, int B, int npos, float* out) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= B * npos) return;
    const int b = i / npos, pos = i % npos;
    U4 r = philox4x32_10((uint32_t)round, (uint32_t)(round >> 32), (uint32_t)b, (uint32_t)pos,
                         (uint32_t)seed, (uint32_t)(seed >> 32));
    out[2 * i + 0] = u01(r.x);
    out[2 * i + 1] = u01(r.y);
}

hipError_t launch_philox(const tabed_cfg& c, uint64_t round, float* out, hipStream_t s) {
    const int count = c.B * (c.gamma + 1);
    launch(nullptr, k_philox, dim3((count + 255) / 256), dim3(256), 0, s, c.seed, round, c.B, c.gamma + 1, out);
    return hipGetLastError();
}

// Window + weights for one sequence, executed by ONE wave (64 lanes).  The window after pushing the nv new
// positions is the newest min(count + nv, h) entries of (old ring entries ++ new entries); every lane loads
// its share of them in parallel (no load depends on a store), lane j sums column j in fp64, the policy
// follows (softmax of 1/e over the n drafts, or arg-min over the 11 candidate mixtures), and only then are the
// new positions stored into the ring.  h = 0 (window ALL): one running fp32 sum per column.  dw = width of
// one distance vector.  PUB: the distances were just published by another workgroup of the same kernel and
// must be read at device scope.  Lanes exchange through two small LDS arrays; LDS operations of one wave
// execute in order, so no barrier is involved.  A few hundred scalars: latency-bound.
struct WindowArgs {
    int n, dw, gamma, h, policy;
    double tau_w, eps;
    uint64_t seed, round;   // policy 3: Philox key and the round the weights are for
    float* ring;
    int32_t* ring_head;
    int32_t* ring_count;
    float* weights;
};

// dev(q): distance q of the sequence's [gamma, dw].  PUB: the weights are published.
template <bool PUB, typename Dev>
__device__ __forceinline__ void window_update(const WindowArgs& a, int b, int lane, Dev dev, int nv,
                                              double* s_part /* [64] */, double* s_x /* [TABED_MAX_N] */) {
    const int n = a.n, dw = a.dw, gamma = a.gamma, h = a.h, policy = a.policy;
    nv = nv < 0 ? 0 : (nv > gamma ? gamma : nv);
    bool empty;
    if (h == 0) {
        int count = a.ring_count[b];
        count = count < 0 ? 0 : count;
        if (lane < dw) {
            float sum = a.ring[(size_t)b * dw + lane];
            for (int i = 0; i < nv; ++i) sum = sum + dev(i * dw + lane);   // fp32, in order
            if (nv > 0) a.ring[(size_t)b * dw + lane] = sum;
            s_x[lane] = (policy == 2) ? (double)sum : (1.0 / fmax((double)sum, a.eps)) / a.tau_w;
        }
        const long long total = (long long)count + nv;
        if (lane == 0 && nv > 0) a.ring_count[b] = total > 0x7fffffffLL ? 0x7fffffff : (int)total;
        empty = (total == 0);
    } else {
        int head = a.ring_head[b], count = a.ring_count[b];
        head = ((head % h) + h) % h;
        count = count < 0 ? 0 : (count > h ? h : count);
        const int new_count = (count + nv < h) ? count + nv : h;
        float* rb = a.ring + (size_t)b * h * dw;
        const int per = 64 / dw;                      // lanes per column (dw <= 16 => per >= 4)
        const int j = lane % dw, t0 = lane / dw;
        double acc = 0.0;
        if (lane < per * dw) {
            for (int r = t0; r < new_count; r += per) {   // r-th newest entry of the new window
                float v;
                if (r < nv) v = dev((nv - 1 - r) * dw + j);
                else        v = rb[(size_t)((((head - 1 - (r - nv)) % h) + h) % h) * dw + j];
                acc += (double)v;
            }
        }
        s_part[lane] = acc;
        __builtin_amdgcn_wave_barrier();
        if (lane < dw) {
            double e = 0.0;
            for (int q = 0; q < per; ++q) e += s_part[q * dw + lane];
            s_x[lane] = (policy == 2) ? e : (1.0 / fmax(e, a.eps)) / a.tau_w;
        }
        if (nv > 0) {                                 // all window loads above are complete: store the new entries
            for (int idx = lane; idx < nv * dw; idx += 64) {
                const int i = idx / dw, jj = idx % dw;
                if (i >= nv - h) rb[(size_t)((head + i) % h) * dw + jj] = dev(i * dw + jj);
            }
            if (lane == 0) {
                a.ring_head[b] = (head + nv) % h;
                a.ring_count[b] = new_count;
            }
        }
        empty = (new_count == 0);
    }
    if (policy == 3 && lane < n) {                     // random weights: E_j = -ln U_j, normalised below
        const U4 r = philox4x32_10((uint32_t)a.round, (uint32_t)(a.round >> 32), (uint32_t)b,
                                   (uint32_t)(gamma + 1 + lane / 4), (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
        const uint32_t x = (lane & 3) == 0 ? r.x : (lane & 3) == 1 ? r.y : (lane & 3) == 2 ? r.z : r.w;
        s_x[lane] = -log(((double)(x >> 8) + 0.5) * (1.0 / 16777216.0));
    }
    __builtin_amdgcn_wave_barrier();
    if (lane < n) {
        float w;
        if (policy == 3) {
            double tot = 0.0;
            for (int q = 0; q < n; ++q) tot += s_x[q];
            w = (float)(s_x[lane] / tot);
        } else if (policy == 1 || empty) {
            w = (float)(1.0 / (double)n);
        } else if (policy == 2) {
            int best = 0;                             // arg-min of the window sums, lowest index on ties
            for (int q = 1; q < dw; ++q) if (s_x[q] < s_x[best]) best = q;
            const double w1 = (double)best / (double)(dw - 1);
            w = (float)(lane == 0 ? 1.0 - w1 : w1);
        } else {
            double xmax = -INFINITY;
            for (int q = 0; q < n; ++q) xmax = fmax(xmax, s_x[q]);
            double Z = 0.0;
            for (int q = 0; q < n; ++q) Z += exp(s_x[q] - xmax);
            w = (float)(exp(s_x[lane] - xmax) / Z);
        }
        if (PUB) publish_store(&a.weights[(size_t)b * n + lane], w);
        else a.weights[(size_t)b * n + lane] = w;
    }
}

__global__ __launch_bounds__(64) void k_weights(WindowArgs a, const float* __restrict__ dev,
                                                const int32_t* __restrict__ n_valid) {
    __shared__ double s_part[64];
    __shared__ double s_x[TABED_MAX_N];
    const int b = blockIdx.x;
    const int nv = (dev != nullptr && n_valid != nullptr) ? n_valid[b] : 0;
    const float* const db = dev + (size_t)b * a.gamma * a.dw;               // (nv = 0: not read)
    window_update<false>(a, b, threadIdx.x, [&](int q) { return db[q]; }, nv, s_part, s_x);
}

static WindowArgs window_args(const tabed_cfg& c, uint64_t round, float* ring, int32_t* ring_head, int32_t* ring_count,
                              float* weights) {
    WindowArgs a;
    a.seed = c.seed; a.round = round;
    a.n = c.n; a.dw = (c.policy == 2) ? TABED_GRID_CANDIDATES : c.n; a.gamma = c.gamma; a.h = c.h; a.policy = c.policy;
    a.tau_w = (double)c.tau_w; a.eps = (double)c.eps;
    a.ring = ring; a.ring_head = ring_head; a.ring_count = ring_count; a.weights = weights;
    return a;
}

hipError_t launch_weights(const tabed_cfg& c, uint64_t round, const float* dev, const int32_t* n_valid, float* ring,
                          int32_t* ring_head, int32_t* ring_count, float* weights, hipStream_t s) {
    ProfScope prof(TABED_K_WEIGHTS, s);
    launch(&prof, k_weights, dim3(c.B), dim3(64), 0, s, window_args(c, round, ring, ring_head, ring_count, weights), dev,
           n_valid);
    return hipGetLastError();
}

// =====================================================================================================
// Ensemble + draft token.
// The LM-head epilogue left, per draft row and per 32-wide vocabulary tile, the tile maximum of the scaled
// logits and the tile sum of exp(scaled logit - tile maximum).  From those alone this kernel gets every
// draft's log-sum-exp and the mass of the mixture q = sum_j w_j q^(j) inside every tile; a sampling row
// therefore reads logits only inside the one tile its uniform falls into.  Every thread loads the partials
// of its own tiles (all drafts) in one burst of independent loads and keeps them in registers, so the kernel
// pays two memory round trips (partials, then the chosen tile) instead of one per reduction.  A greedy row needs
// the arg-max of q over the whole vocabulary: its row is split over gridDim.x workgroups and the last one
// to arrive merges the candidates (lowest index wins ties, so arrival order does not matter).
// =====================================================================================================
struct SampleArgs {
    int V, n, B, gamma, pos, NT, C2, TS;
    int S;                // token tree: siblings per position; 0: this launch draws the trunk token
    const int32_t* trunk; // token tree: trunk tokens [B,gamma] (a greedy row's siblings skip the trunk's token)
    uint64_t seed, round;
    const float* logits;  // [B,n,V] of this position
    const float* pm;      // [B*n,NT]
    const float* ps;      // [B*n,NT]
    const float* weights;
    const float* temperature;
    const float* u_draft;
    double* draft_lse;
    int32_t* draft_tokens;
    float* draft_q;
    uint8_t* flags;
    Top2Rec* cand;        // [B][C2] trunk token
    Top3Rec* cand3;       // [S][B][C2] siblings
    uint32_t* tickets;    // siblings: S counters of a sequence, B * TS apart
};

// TI = tiles per thread, a compile-time bound with NT <= kBlock * TI, so that every phase issues all of its
// loads before the first use and keeps its tile values in registers.  N = number of drafts when it is known
// at compile time (0 = run time): then the partials are read ONCE, each thread keeping the n*TI terms
// ps*exp(pm - m_j) of its own run of tiles in registers for both the log-sum-exp and the tile masses.
template <int TI, int N, int THR = kBlock>
__global__ __launch_bounds__(THR) void k_sample(SampleArgs a) {
    constexpr int NWV = THR / kWave;
    static_assert(N == 0 || THR == kBlock, "the sums of the single pass are those of four waves");
    const int c = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int b = (int)blockIdx.x + c;                           // (blockIdx.x + c) % B, c < 8
    while (b >= a.B) b -= a.B;
    const int n = (N > 0) ? N : a.n, NT = a.NT, V = a.V;
    const int sib = a.S > 0 ? (int)blockIdx.z + 1 : 0;     // 0: the trunk token; siblings of a position in one launch
    // Workgroup 0 of a sequence always has work, so its temperature load overlaps the loads below; the
    // other workgroups only exist for greedy rows and leave at once otherwise.
    const float T = a.temperature[b];
    if (c != 0 && T > 0.f) return;

    __shared__ float s_m[TABED_MAX_N];    // row maximum of scaled logits
    __shared__ double s_S[TABED_MAX_N];   // sum_v exp(scaled - max)
    __shared__ double s_c[TABED_MAX_N];   // w_j / S_j
    __shared__ float s_cf[TABED_MAX_N];
    __shared__ int s_first[NWV], s_lastw[NWV], s_tile, s_last;
    __shared__ double s_prefix;
    __shared__ Top3 s_top[NWV];
    __shared__ double s_term[TABED_MAX_N][kTileV];
    __shared__ float s_wm[NWV][TABED_MAX_N];
    __shared__ double s_wsum[NWV][TABED_MAX_N];
    __shared__ double s_wtot[NWV][8];        // wave totals of the tile-mass scan, per chunk row
    constexpr int kMaxTiles = THR * TI, kMaxListed = 64;                // greedy rows: tiles that may hold the arg-max
    __shared__ uint32_t s_live[(kMaxTiles + 31) / 32];
    __shared__ int s_list[kMaxListed], s_count;
    __shared__ ArgMax s_wtop[NWV];
    __shared__ float s_reach;

    const float* pmb = a.pm + (size_t)b * n * NT;      // partials of this sequence: [n][NT]
    const float* psb = a.ps + (size_t)b * n * NT;
    // the trunk token goes to [B,gamma]; sibling s of a token tree to [B,gamma,S] and has a Philox block of its own
    const size_t out_idx = (sib == 0) ? (size_t)b * a.gamma + a.pos
                                      : ((size_t)b * a.gamma + a.pos) * a.S + (sib - 1);
    const float wj = (tid < n) ? a.weights[(size_t)b * n + tid] : 0.f;
    const float u = a.u_draft ? a.u_draft[out_idx]
                              : tabed_uniform(a.seed, a.round, (uint32_t)b, (uint32_t)a.pos + (uint32_t)sib * kSiblingStride, 0);
    // greedy siblings: the largest entries other than the trunk's token; sibling s takes the s-th of them
    const int taken = (sib > 0) ? a.trunk[(size_t)b * a.gamma + a.pos] : -1, rank = (sib > 0) ? sib - 1 : 0;

    // Which tiles a thread owns.  TI = 1: tile tid.  Else TI/4 chunks of 4 consecutive tiles, chunk q*256 + tid for
    // q < TI/4 -- every load is then 16 bytes and a wave's load is one contiguous kilobyte.  (A run of TI = 20 tiles per
    // thread read element by element looked up 40 lines an instruction: 65 us at V = 128256 with 8 drafts, 64 sequences.)
    constexpr bool CHUNKED = (TI >= 4);
    constexpr int TPC = CHUNKED ? 4 : TI;              // tiles per chunk
    constexpr int Q = TI / TPC;                        // chunks per thread
    auto tile_of = [&](int i) { return CHUNKED ? ((i / 4) * THR + tid) * 4 + (i & 3) : tid * TI + i; };

    // this thread's tiles of one draft's partials: maxima and, with WITH_SUMS, sums
    auto load_tiles = [&](int j, float (&m)[TI], float (&sum)[TI], auto with_sums) {
        const float* pr = pmb + (size_t)j * NT;
        const float* sr = psb + (size_t)j * NT;
        if (CHUNKED && (NT & 3) == 0) {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int t = tile_of(4 * q);
                float4 m4 = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY), s4 = make_float4(0.f, 0.f, 0.f, 0.f);
                if (t < NT) {
                    m4 = *reinterpret_cast<const float4*>(pr + t);
                    if (with_sums.value) s4 = *reinterpret_cast<const float4*>(sr + t);
                }
                m[4 * q] = m4.x; m[4 * q + 1] = m4.y; m[4 * q + 2] = m4.z; m[4 * q + 3] = m4.w;
                if (with_sums.value) { sum[4 * q] = s4.x; sum[4 * q + 1] = s4.y; sum[4 * q + 2] = s4.z; sum[4 * q + 3] = s4.w; }
            }
        } else {
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                const int t = tile_of(i);
                m[i] = t < NT ? pr[t] : -INFINITY;
                if (with_sums.value) sum[i] = t < NT ? sr[t] : 0.f;
            }
        }
    };
    float uu[(N > 0) ? N : 1][TI];                     // single pass: terms of this thread's tiles, all drafts
    float pmv[(N > 0) ? N : 1][TI];                    // and their maxima
    double lse_mine = 0.0;
    if (N > 0) {
        // ---- single pass over the partials of every draft
        float psv[(N > 0) ? N : 1][TI];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            load_tiles(j, pmv[j], psv[j], std::true_type{});
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            float ml = -INFINITY;
#pragma unroll
            for (int i = 0; i < TI; ++i) ml = fmaxf(ml, pmv[j][i]);
            ml = wave_max(ml);
            if (lane == 0) s_wm[wave][j] = ml;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const float M = fmaxf(fmaxf(s_wm[0][j], s_wm[1][j]), fmaxf(s_wm[2][j], s_wm[3][j]));
            float sl = 0.f;
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                uu[j][i] = (psv[j][i] > 0.f) ? psv[j][i] * __expf(pmv[j][i] - M) : 0.f;
                sl += uu[j][i];
            }
            const double S = wave_sum((double)sl);         // TI terms in fp32, fp64 across lanes and waves
            if (lane == 0) s_wsum[wave][j] = S;
        }
        __syncthreads();
        if (tid < N) {                                     // thread j: everything the later phases need of draft j
            const int j = tid;
            const float M = fmaxf(fmaxf(s_wm[0][j], s_wm[1][j]), fmaxf(s_wm[2][j], s_wm[3][j]));
            const double S = (s_wsum[0][j] + s_wsum[1][j]) + (s_wsum[2][j] + s_wsum[3][j]);
            s_m[j] = M;
            s_S[j] = S;
            s_c[j] = (double)wj / S;
            s_cf[j] = (float)s_c[j];
            lse_mine = (double)M + log(S);                 // stored after the barrier below
        }
    } else {
        // ---- per-draft log-sum-exp: one wave per draft row, lanes strided over the row's tiles
        constexpr int TL = TI * NWV;        // tiles per lane when one wave covers a whole row
        for (int j = wave; j < n; j += NWV) {
            float pmv[TL], psv[TL];
#pragma unroll
            for (int i = 0; i < TL; ++i) {
                const int t = lane + i * kWave;
                pmv[i] = t < NT ? pmb[(size_t)j * NT + t] : -INFINITY;
                psv[i] = t < NT ? psb[(size_t)j * NT + t] : 0.f;
            }
            float ml = -INFINITY;
#pragma unroll
            for (int i = 0; i < TL; ++i) ml = fmaxf(ml, pmv[i]);
            const float M = wave_max(ml);
            float sl = 0.f;
#pragma unroll
            for (int i = 0; i < TL; ++i) sl += (psv[i] > 0.f) ? psv[i] * __expf(pmv[i] - M) : 0.f;
            const double S = wave_sum((double)sl);
            if (lane == 0) {
                s_m[j] = M;
                s_S[j] = S;
                if (c == 0 && sib == 0) a.draft_lse[((size_t)a.pos * a.B + b) * n + j] = (double)M + log(S);
            }
        }
    }
    const bool greedy = !(T > 0.f);
    const float invT = greedy ? 1.f : 1.f / T;
    __syncthreads();
    if (N > 0) {
        if (tid < N && c == 0 && sib == 0) a.draft_lse[((size_t)a.pos * a.B + b) * n + tid] = lse_mine;
    } else {
        if (tid < n) {
            s_c[tid] = (double)wj / s_S[tid];
            s_cf[tid] = (float)s_c[tid];
        }
        __syncthreads();
    }

    const float* rows = a.logits + (size_t)b * n * V;

    if (!greedy) {
        // ---- tile masses of the mixture: thread tid owns tiles [tid*TI, tid*TI + TI), kept in registers
        double mt[TI];
#pragma unroll
        for (int i = 0; i < TI; ++i) mt[i] = 0.0;
        double Z = 0.0;
        if (N > 0) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const double cj = s_c[j];
                Z += cj * s_S[j];
#pragma unroll
                for (int i = 0; i < TI; ++i) mt[i] += cj * (double)uu[j][i];
            }
        } else {
#pragma unroll 2
            for (int j = 0; j < n; ++j) {
                float pmv[TI], psv[TI];
                load_tiles(j, pmv, psv, std::true_type{});
                const double cj = s_c[j];
                const float mj = s_m[j];
                Z += cj * s_S[j];
#pragma unroll
                for (int i = 0; i < TI; ++i)
                    if (psv[i] > 0.f) mt[i] += cj * (double)(psv[i] * __expf(pmv[i] - mj));
            }
        }
        // ---- prefix over the tile masses in tile order.  Chunk q of thread tid has key q*256 + tid; keys
        //      order the chunks along the vocabulary.  One wave scan per chunk row, one barrier.
        double cs[Q], cinc[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            cs[q] = 0.0;
#pragma unroll
            for (int e = 0; e < TPC; ++e) cs[q] += mt[q * TPC + e];
            cinc[q] = wave_inclusive_scan(cs[q]);
            if (lane == 63) s_wtot[wave][q] = cinc[q];
        }
        __syncthreads();
        const double target = (double)u * Z;
        double excl[Q];
        int first_key = 0x7fffffff, last_key = -1;
        {
            double rowbase = 0.0, wt[NWV][Q];              // all totals requested together (one after the other 1 us at V = 152064)
#pragma unroll
            for (int w = 0; w < NWV; ++w)
#pragma unroll
                for (int q = 0; q < Q; ++q) wt[w][q] = s_wtot[w][q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                double before = rowbase;
#pragma unroll
                for (int w = 0; w < NWV - 1; ++w) before = (w < wave) ? before + wt[w][q] : before;
                excl[q] = before + (cinc[q] - cs[q]);
                if (cs[q] > 0.0) {
                    if (first_key == 0x7fffffff && excl[q] + cs[q] > target) first_key = q * THR + tid;
                    last_key = q * THR + tid;
                }
                double row = wt[0][q];
#pragma unroll
                for (int w = 1; w < NWV; ++w) row += wt[w][q];
                rowbase += row;
            }
        }
        const int key = block_pick_key<NWV>(first_key, last_key, s_first, s_lastw);   // -1 only if every mass is zero
        if (key < 0) {
            if (tid == 0) {
                a.draft_tokens[out_idx] = 0;
                a.draft_q[out_idx] = 0.f;
                a.flags[out_idx] = (uint8_t)(TABED_FLAG_SAMPLE_MARGIN | TABED_FLAG_DEGENERATE);
            }
            return;
        }
        if (tid == (key & (THR - 1))) {
            const int qs = key / THR;
            double P = 0.0, Plast = 0.0;
            int istar = -1, ilast = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (q == qs) {
                    P = excl[q]; Plast = P; ilast = q * TPC;
#pragma unroll
                    for (int e = 0; e < TPC; ++e) {
                        const int i = q * TPC + e;
                        if (istar < 0) {
                            if (mt[i] > 0.0) { ilast = i; Plast = P; }
                            if (P + mt[i] > target) istar = i;
                            else P += mt[i];
                        }
                    }
                }
            }
            if (istar < 0) { istar = ilast; P = Plast; }
            s_tile = tile_of(istar);
            s_prefix = P;
        }
        __syncthreads();
        // ---- the tile's logits: thread (draft j, lane v) -> one round trip for all drafts, summed by wave 0
        {
            const int vl = tid & (kTileV - 1), v = s_tile * kTileV + vl;
            for (int j = tid / kTileV; j < n; j += THR / kTileV)
                s_term[j][vl] = (v < V) ? s_c[j] * (double)__expf(rows[(size_t)j * V + v] * invT - s_m[j]) : 0.0;
        }
        __syncthreads();
        if (tid >= kWave) return;
        const int v = s_tile * kTileV + lane;
        double f = 0.0;
        if (lane < kTileV)
            for (int j = 0; j < n; ++j) f += s_term[j][lane];
        const double inc = wave_inclusive_scan(f);
        const double cdf = s_prefix + inc;
        const unsigned long long cross = __ballot(cdf > target && f > 0.0);
        const unsigned long long live = __ballot(f > 0.0);
        int pick;
        uint32_t flag = 0;
        if (cross) pick = __ffsll((long long)cross) - 1;
        else if (live) { pick = 63 - __clzll((long long)live); flag = TABED_FLAG_SAMPLE_MARGIN | TABED_FLAG_DEGENERATE; }
        else { pick = 0; flag = TABED_FLAG_SAMPLE_MARGIN | TABED_FLAG_DEGENERATE; }
        if (lane == pick) {
            const double tol = (double)kMargin * Z;
            if (fabs(cdf - target) < tol && v + 1 < V) flag |= TABED_FLAG_SAMPLE_MARGIN;
            if (v > 0 && fabs((cdf - f) - target) < tol) flag |= TABED_FLAG_SAMPLE_MARGIN;
            a.draft_tokens[out_idx] = v < V ? v : V - 1;
            a.draft_q[out_idx] = (float)f;
            a.flags[out_idx] = (uint8_t)flag;
        }
        return;
    }

    // ---- greedy row: arg-max (with runner-up) of the mixture.  A tile's partials bound the mixture inside it,
    //      q(v) <= sum_j (w_j / S_j) exp(pm_jt - m_j); the tile with the largest bound is evaluated first, and only tiles whose
    //      bound reaches its maximum (less a margin far above the rounding of either side and the 1e-6 of the near-tie
    //      flag) can hold the arg-max or a runner-up that matters.  With language-model logits these are a handful: one
    //      workgroup evaluates them, its siblings leave.  If there are more (flat distributions) the row's workgroups
    //      (at most kMaxGreedyChunks: every one of them repeats the pass over the row's partials) share the walk over the
    //      vocabulary and read the surviving tiles only.
    float ub[TI];
#pragma unroll
    for (int i = 0; i < TI; ++i) ub[i] = 0.f;
    if (N > 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const float cj = s_cf[j], mj = s_m[j];
#pragma unroll
            for (int i = 0; i < TI; ++i) ub[i] += cj * __expf(pmv[j][i] - mj);
        }
    } else {
#pragma unroll 2
        for (int j = 0; j < n; ++j) {
            const float cj = s_cf[j], mj = s_m[j];
            float pj[TI];
            load_tiles(j, pj, pj, std::false_type{});
#pragma unroll
            for (int i = 0; i < TI; ++i) ub[i] += cj * __expf(pj[i] - mj);
        }
    }
    ArgMax top{-INFINITY, 0x7fffffff};
#pragma unroll
    for (int i = 0; i < TI; ++i)
        if (tile_of(i) < NT) top = argmax_merge(top, ArgMax{ub[i], tile_of(i)});
    top = wave_argmax(top);
    if (lane == 0) s_wtop[wave] = top;
    for (int i = tid; i < (kMaxTiles + 31) / 32; i += THR) s_live[i] = 0u;
    if (tid == 0) s_count = 0;
    __syncthreads();
    // (one record after the other cost a greedy row 0.3 us, of 10 to 18 a draft step; in pairs, the sampling rows 0.1 us: the compiler
    // then allots their part of the kernel other registers)
    ArgMax first = s_wtop[lane & (NWV - 1)];
    first = argmax_dpp_step<kDppXor1>(first);
    first = argmax_dpp_step<kDppXor2>(first);
    if (NWV > 4) first = argmax_dpp_step<kDppHalfMirror>(first);           // (lane ^ 7: the other four)
    first = argmax_at(first, 0);
    const int t0 = first.i;
    // the mixture at one vocabulary entry, drafts in order, and whether it may be drawn
    auto mixture = [&](int v) {
        float q = 0.f;
        if (N > 0) {
            float x[(N > 0) ? N : 1];
#pragma unroll
            for (int j = 0; j < N; ++j) x[j] = rows[(size_t)j * V + v];
#pragma unroll
            for (int j = 0; j < N; ++j) q += s_cf[j] * __expf(x[j] * invT - s_m[j]);
        } else {
#pragma unroll 8
            for (int j = 0; j < n; ++j) q += s_cf[j] * __expf(rows[(size_t)j * V + v] * invT - s_m[j]);
        }
        return q;
    };
    auto may_draw = [&](int v) { return v < V && v != taken; };
    if (wave == 0) {
        const int v = t0 * kTileV + (lane & 31);
        const float q = (lane < kTileV && t0 < NT && may_draw(v)) ? mixture(v) : -INFINITY;
        Top3 t = top3_empty();
        if (q > -INFINITY) t = Top3{q, v, -INFINITY, 0x7fffffff, -INFINITY};
        t = wave_top3(t);
        const float reach = (rank == 0) ? t.v1 : t.v2;     // at least rank + 1 entries reach this
        if (lane == 0) s_reach = (reach > 0.f) ? reach * (1.f - 3e-5f) : -INFINITY;
    }
    __syncthreads();
    const float reach = s_reach;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
        const int t = tile_of(i);
        if (t < NT && !(ub[i] < reach)) {
            atomicOr(&s_live[t >> 5], 1u << (t & 31));
            const int at = atomicAdd(&s_count, 1);
            if (at < kMaxListed) s_list[at] = t;
        }
    }
    __syncthreads();
    const int listed = s_count;
    Top3 best = top3_empty();
    const bool few = (listed <= kMaxListed);              // the same in every workgroup of the row
    if (few) {
        if (c != 0) return;
        // a half-wave takes TB tiles at a time, all drafts of all of them requested together (64 tiles one after the other: 11 us)
        auto evaluate = [&](auto tb) {
            constexpr int TB = tb.value, kApart = THR / kTileV;
            for (int a0 = tid >> 5; a0 < listed; a0 += TB * kApart) {
                int v[TB];
                float q[TB];
#pragma unroll
                for (int b = 0; b < TB; ++b) {
                    v[b] = s_list[min(a0 + b * kApart, listed - 1)] * kTileV + (tid & 31);
                    q[b] = 0.f;
                }
                if (N > 0) {
                    float x[TB][(N > 0) ? N : 1];
#pragma unroll
                    for (int b = 0; b < TB; ++b)
#pragma unroll
                        for (int j = 0; j < N; ++j) x[b][j] = rows[(size_t)j * V + min(v[b], V - 1)];
#pragma unroll
                    for (int b = 0; b < TB; ++b)
#pragma unroll
                        for (int j = 0; j < N; ++j) q[b] += s_cf[j] * __expf(x[b][j] * invT - s_m[j]);
                } else {
#pragma unroll 4
                    for (int j = 0; j < n; ++j)
#pragma unroll
                        for (int b = 0; b < TB; ++b) q[b] += s_cf[j] * __expf(rows[(size_t)j * V + min(v[b], V - 1)] * invT - s_m[j]);
                }
#pragma unroll
                for (int b = 0; b < TB; ++b)
                    if (a0 + b * kApart < listed && may_draw(v[b])) best = top3_push(best, q[b], v[b]);
            }
        };
        if (listed <= THR / kTileV) evaluate(std::integral_constant<int, 1>{});
        else evaluate(std::integral_constant<int, 4>{});
    } else {
        for (int cb = c * kChunkV; cb < V; cb += a.C2 * kChunkV) {
            constexpr int UG = kChunkV / (THR * 4);        // groups of four entries a thread
            float q[UG][4];
            bool live[UG];
            int at[UG];
#pragma unroll
            for (int u = 0; u < UG; ++u) {
                const int v = cb + (u * THR + tid) * 4, t = min(v, V - 1) / kTileV;
                live[u] = (s_live[t >> 5] >> (t & 31)) & 1u;
                at[u] = live[u] ? group_at(v, V) : 0;      // (a group that cannot matter costs one shared line: behind a branch,
                                                           // every load waited for the one before it, 9 us a chunk)
#pragma unroll
                for (int e = 0; e < 4; ++e) q[u][e] = 0.f;
            }
            constexpr int JB = 4;                          // draft rows requested together
            for (int j0 = 0; j0 < n; j0 += JB) {
                float4 x[JB][UG];
#pragma unroll
                for (int jj = 0; jj < JB; ++jj)            // past the last draft: re-read, not used
#pragma unroll
                    for (int u = 0; u < UG; ++u)            // (more than kMaxListed tiles: not a short row)
                        x[jj][u] = load_group(rows + (size_t)min(j0 + jj, n - 1) * V, at[u]);
#pragma unroll
                for (int jj = 0; jj < JB; ++jj)
                    if (j0 + jj < n) {
                        const float cj = s_cf[j0 + jj], mj = s_m[j0 + jj];
#pragma unroll
                        for (int u = 0; u < UG; ++u)
#pragma unroll
                            for (int e = 0; e < 4; ++e) q[u][e] += cj * __expf(f4get(x[jj][u], e) * invT - mj);
                    }
            }
#pragma unroll
            for (int u = 0; u < UG; ++u) {
                const int v = cb + (u * THR + tid) * 4;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (live[u] && at[u] + e >= v && may_draw(at[u] + e)) best = top3_push(best, q[u][e], at[u] + e);
            }
        }
    }
    best = wave_top3(best);
    if (lane == 0) s_top[wave] = best;
    __syncthreads();
    if (!few && tid == 0) {
        Top3 t = s_top[0];
        for (int w = 1; w < NWV; ++w) t = top3_merge(t, s_top[w]);
        if (sib == 0) {
            Top2Rec* rec = &a.cand[(size_t)b * a.C2 + c];
            publish_store(&rec->v1, t.v1);
            publish_store(&rec->i1, t.i1);
            publish_store(&rec->v2, t.v2);
        } else {
            Top3Rec* rec = &a.cand3[((size_t)rank * a.B + b) * a.C2 + c];
            publish_store(&rec->v1, t.v1);
            publish_store(&rec->i1, t.i1);
            publish_store(&rec->v2, t.v2);
            publish_store(&rec->i2, t.i2);
            publish_store(&rec->v3, t.v3);
        }
    }
    Top3 t = top3_empty();
    if (few) {
        if (tid >= kWave) return;
        if (lane < NWV) t = s_top[lane];
    } else {
        publish_barrier();                                 // the candidate's stores are acknowledged
        if (tid == 0) s_last = arrive(&a.tickets[((size_t)rank * a.B + b) * a.TS], (uint32_t)a.C2) ? 1 : 0;
        __syncthreads();
        if (!s_last || tid >= kWave) return;
        for (int cc = lane; cc < a.C2; cc += kWave) {
            if (sib == 0) {
                const Top2Rec* r = &a.cand[(size_t)b * a.C2 + cc];
                t = top3_merge(t, Top3{published_load(&r->v1), published_load(&r->i1), published_load(&r->v2), 0x7ffffffe, -INFINITY});
            } else {
                const Top3Rec* r = &a.cand3[((size_t)rank * a.B + b) * a.C2 + cc];
                t = top3_merge(t, Top3{published_load(&r->v1), published_load(&r->i1), published_load(&r->v2), published_load(&r->i2),
                                       published_load(&r->v3)});
            }
        }
    }
    t = wave_top3(t);
    if (lane != 0) return;
    const float won = (rank == 0) ? t.v1 : t.v2, next = (rank == 0) ? t.v2 : t.v3;
    const int at = (rank == 0) ? t.i1 : t.i2;
    const int y = (at >= 0 && at < V) ? at : 0;
    double f = 0.0;
#pragma unroll 8
    for (int j = 0; j < n; ++j) f += s_c[j] * (double)__expf(rows[(size_t)j * V + y] * invT - s_m[j]);
    uint32_t flag = 0;
    if (V > 1 + sib && (won - next) < kMargin * fabsf(won)) flag |= TABED_FLAG_SAMPLE_MARGIN;
    a.draft_tokens[out_idx] = y;
    a.draft_q[out_idx] = (float)f;
    a.flags[out_idx] = (uint8_t)flag;
}

// S = 0: the trunk token of Alg. 1 (Sample step).  S >= 1 (token tree): the S siblings of the position in one launch, from
// the same softmax partials; the output arrays are then the [B,gamma,S] sibling arrays.
static hipError_t launch_sample_any(const tabed_cfg& c, const WsLayout& L, char* ws, uint64_t round, int pos,
                                    const float* logits, const float* weights, const float* temperature,
                                    const float* u_draft, double* draft_lse, int32_t* draft_tokens, float* draft_q,
                                    uint8_t* flags, int S, const int32_t* trunk, hipStream_t s) {
    ProfScope prof(TABED_K_SAMPLE, s);
    SampleArgs a;
    a.V = c.V; a.n = c.n; a.B = c.B; a.gamma = c.gamma; a.pos = pos; a.NT = L.NT; a.C2 = L.C2; a.TS = L.TS;
    a.S = S; a.trunk = trunk;
    a.seed = c.seed; a.round = round;
    a.logits = logits;
    a.pm = reinterpret_cast<const float*>(ws + L.off_pm);
    a.ps = reinterpret_cast<const float*>(ws + L.off_ps);
    a.weights = weights; a.temperature = temperature; a.u_draft = u_draft;
    a.draft_lse = draft_lse; a.draft_tokens = draft_tokens; a.draft_q = draft_q; a.flags = flags;
    a.cand = reinterpret_cast<Top2Rec*>(ws + L.off_cand);
    // siblings: the counters and the room of the tree passes, which run after them (3 C2 <= NSEG wherever a row is shared)
    a.cand3 = reinterpret_cast<Top3Rec*>(ws + L.off_tseg);
    a.tickets = reinterpret_cast<uint32_t*>(ws + L.off_tickets) + (S > 0 ? 3 : 0) * (size_t)c.B * L.TS;
    const int ti = (L.NT + kBlock - 1) / kBlock;
    const bool wide = (ti > 8 && c.n > 4) || ti > 20;
    // Eight waves of 250 registers: one workgroup a compute unit, so that half as many share a greedy row where all would not fit at once
    // (draft steps, d = 64, with eight / with four a greedy row: V = 128256, 8 drafts, 33 greedy sequences 72.3 / 60.4 us, 64 103.5 / 85.6, 64 of which
    // half are greedy 97.1 / 82.3; 70001, 5 drafts, 33 70.2 / 59.3; 190001, 3 drafts, 33 93.2 / 80.2).
    if (wide && ti <= 24 && (long)c.B * a.C2 > 256) a.C2 = (a.C2 + 1) / 2;
    // The first workgroups of the rows, which do the work of sampling rows alone, on every XCD in turn (all on one with the row's
    // workgroups next to each other: V = 128256, 8 drafts, 64 sampling rows, a draft step with d = 256 128 us, 103 so), and a greedy
    // row's on different ones.
    const dim3 grid(c.B, a.C2, S > 0 ? S : 1);
    // single-pass instantiations: compile-time draft counts whose n*TI terms (x3 registers) fit a 512-register wave
#define TABED_LAUNCH_SAMPLE_N(TI_, N_) launch(&prof, k_sample<TI_, N_>, grid, dim3(kBlock), 0, s, a)
    // Vocabularies of more than 65536 with more than four drafts, or of more than 163840: eight waves, since one workgroup a row
    // reads all of its partials twice (sampler at V = 128256, 8 drafts, 64 sequences, half of them greedy: 37 us with four waves and
    // all rows' first workgroups on one XCD, 27; draft steps of small batches: 8 drafts of 70000 34.9 / 30.7 us, 16 of 150001 58.6 / 44.9,
    // 8 of 190001 68 / 49; rows of equal logits, 4 sequences of 8 drafts 64 / 52).
#define TABED_LAUNCH_SAMPLE(TI_, ALLOW8_)                                       \
    do {                                                                        \
        if (c.n == 1) TABED_LAUNCH_SAMPLE_N(TI_, 1);                            \
        else if (c.n == 2) TABED_LAUNCH_SAMPLE_N(TI_, 2);                       \
        else if (c.n == 3) TABED_LAUNCH_SAMPLE_N(TI_, 3);                       \
        else if (c.n == 4) TABED_LAUNCH_SAMPLE_N(TI_, 4);                       \
        else if (!ALLOW8_) return hipErrorInvalidValue;                         \
        else if (c.n == 5) TABED_LAUNCH_SAMPLE_N(TI_, (ALLOW8_ ? 5 : 1));       \
        else if (c.n == 8) TABED_LAUNCH_SAMPLE_N(TI_, (ALLOW8_ ? 8 : 1));       \
        else TABED_LAUNCH_SAMPLE_N(TI_, (ALLOW8_ ? 0 : 1));                     \
    } while (0)
    if (ti <= 1) TABED_LAUNCH_SAMPLE(1, true);
    else if (ti <= 4) TABED_LAUNCH_SAMPLE(4, true);
    else if (ti <= 8) TABED_LAUNCH_SAMPLE(8, true);
    else if (!wide) TABED_LAUNCH_SAMPLE(20, false);
    else if (ti <= 24) launch(&prof, k_sample<12, 0, 512>, grid, dim3(512), 0, s, a);
    else if (ti <= 32) TABED_LAUNCH_SAMPLE_N(32, 0);   // (eight waves of 16 tiles a thread spill)
    else return hipErrorInvalidValue;              // V > 262144: validate_cfg rejects it before this point
#undef TABED_LAUNCH_SAMPLE_N
#undef TABED_LAUNCH_SAMPLE
    return hipGetLastError();
}

hipError_t launch_sample(const tabed_cfg& c, const WsLayout& L, char* ws, uint64_t round, int pos,
                         const float* logits, const float* weights, const float* temperature,
                         const float* u_draft, double* draft_lse, int32_t* draft_tokens, float* draft_q,
                         uint8_t* flags, hipStream_t s) {
    return launch_sample_any(c, L, ws, round, pos, logits, weights, temperature, u_draft, draft_lse, draft_tokens,
                             draft_q, flags, 0, nullptr, s);
}

// Token tree: the width-1 siblings of position pos.  Uses the softmax partials the LM head of this position left in the
// workspace.  One launch for all of them (one each took 5.7 us a sibling).
hipError_t launch_siblings(const tabed_cfg& c, const WsLayout& L, char* ws, uint64_t round, int pos, int width,
                           const float* logits, const int32_t* draft_tokens, const float* weights,
                           const float* temperature, const float* u_sib, int32_t* sib_tokens, float* sib_q,
                           uint8_t* sib_flags, hipStream_t s) {
    static_assert(TABED_MAX_TREE_WIDTH == 3, "greedy siblings are the two largest entries besides the trunk's");
    return launch_sample_any(c, L, ws, round, pos, logits, weights, temperature, u_sib, nullptr, sib_tokens, sib_q, sib_flags,
                             width - 1, draft_tokens, s);
}

// =====================================================================================================
// Target statistics and per-draft KL sums.
// Grid (chunk, position i <= gamma, sequence b).  Each workgroup reads its chunk of the target row once,
// and for i < gamma the same chunk of the n draft rows once -- all loads issued before the first use --
// and leaves a record
//   { m_c = max scaled target logit, Z_c = sum exp(st - m_c), arg-max of the raw row,
//     A_jc = sum exp(st - m_c) * (st - s_j)  for every draft j }.
// Since KL(p || q_j) = sum_v p (st - s_j) - lse_p + lse_j, the records of a row combine exactly (fp64, chunk
// order) in the kernel that follows.  N is the number of drafts when known at compile time (0 = run time).
// Two-draft grid policy with KL: the same pass leaves, instead of the A_jc, the sums of the 11 candidate mixtures
//   A_kc = sum exp(st - m_c) * (st - log mix_k),   mix_k = (1 - k/10) q_1 + (k/10) q_2,   KL(p || mix_k) = A_k / Z - lse_p,
// so that the distances of that policy cost no pass of their own either.
// =====================================================================================================
struct StatsArgs {
    int V, n, B, gamma, C3, RS;
    int with_drafts;      // 0: only the target-row part of the records (distances come from dist_chunk)
    int grid;             // 1 (two drafts): the A sums are those of the 11 candidate mixtures, not of the drafts
    const float* target;
    const float* dlogits;
    const double* dlse;   // [gamma,B,n]; read only for the mixtures
    const float* temperature;
    double* stats;
};

template <int U, int N>
__device__ __forceinline__ void stats_chunk(const StatsArgs& a, int c, int i, int b) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int V = a.V, n = (N > 0) ? N : a.n, gamma = a.gamma;
    const float T = a.temperature[b];
    const float invT = (T > 0.f) ? 1.f / T : 1.f;

    __shared__ float s_redf[kWavesPerBlock];
    __shared__ double s_redd[kWavesPerBlock];
    __shared__ ArgMax s_am[kWavesPerBlock];
    __shared__ double s_A[kWavesPerBlock][TABED_MAX_N];
    __shared__ float s_qhi[2], s_qoml[2];                // the two drafts' log-sum-exp as fp32 head + (1 - tail)

    const float* trow = a.target + ((size_t)b * (gamma + 1) + i) * V;
    const float* qbase = a.dlogits + (((size_t)i * a.B + b) * n) * V;   // only dereferenced when i < gamma
    const int cb = c * (kBlock * 4 * U);
    const bool inside = cb + kBlock * 4 * U <= V;
    const bool drafts = (i < gamma) && a.with_drafts;
    const bool grid = (N == 2) && drafts && a.grid;
    if (N == 2 && grid && tid < 2) {                     // published by the barriers of the maximum below
        const double l = a.dlse[((size_t)i * a.B + b) * 2 + tid];
        const float hi = (float)l;
        s_qhi[tid] = hi;
        s_qoml[tid] = (float)(1.0 - (l - (double)hi));
    }

    float4 tx[U];
    float4 dx[(N > 0) ? N : 1][U];
    auto v = [&](int u) { return cb + (u * kBlock + tid) * 4; };
    auto at = [&](int u) { return group_at(v(u), V); };
    with_row_loads(V, [&](auto load) {
#pragma unroll
        for (int u = 0; u < U; ++u) tx[u] = load(trow, at(u));
        if (N > 0 && drafts) {
#pragma unroll
            for (int j = 0; j < N; ++j)
#pragma unroll
                for (int u = 0; u < U; ++u) dx[j][u] = load(qbase + (size_t)j * V, at(u));
        }
    });
    if (!inside) {                                       // (a draft's element counts where the target's does: ex > 0)
#pragma unroll
        for (int u = 0; u < U; ++u) mask_group(tx[u], at(u), v(u));
    }

    float st[U * 4], ex[U * 4];
    ArgMax am{-INFINITY, 0x7fffffff};
    float tmax = -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float xe = f4get(tx[u], e);
            if (at(u) + e >= v(u) && at(u) + e < V) am = argmax_merge(am, ArgMax{xe, at(u) + e});
            st[u * 4 + e] = xe * invT;
            tmax = fmaxf(tmax, st[u * 4 + e]);
        }
    }
    const float mc = block_max(tmax, s_redf);
    float zf = 0.f;
#pragma unroll
    for (int k = 0; k < U * 4; ++k) {
        ex[k] = (st[k] > -INFINITY) ? __expf(st[k] - mc) : 0.f;
        zf += ex[k];
    }
    const double Zw = wave_sum((double)zf);
    if (lane == 0) s_redd[wave] = Zw;
    am = wave_argmax(am);
    if (lane == 0) s_am[wave] = am;

    if (N == 2 && grid) {
        // both drafts' probabilities of this thread's elements, then one candidate mixture at a time.  The sums are
        // taken about the chunk maximum (st - m_c <= 0 where exp(st - m_c) matters) and m_c Z_c is added back in
        // fp64 when the record is written.  Bare v_log_f32 (log2): its ~1e-7 relative error is random per element
        // and averages out under the sum; a mixture below the normal range only occurs where p is negligible too.
        float q0[U * 4], q1[U * 4];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a0 = f4get(dx[0][u], e), a1 = f4get(dx[(N > 1) ? 1 : 0][u], e);
                const float p0 = (a0 > -INFINITY) ? __expf(a0 * invT - s_qhi[0]) * s_qoml[0] : 0.f;
                const float p1 = (a1 > -INFINITY) ? __expf(a1 * invT - s_qhi[1]) * s_qoml[1] : 0.f;
                q0[u * 4 + e] = p0;
                q1[u * 4 + e] = p1;
            }
        constexpr int NC = TABED_GRID_CANDIDATES;
        float tl[U * 4];                                   // log2 of exp(st - m_c), shared by the candidates
#pragma unroll
        for (int x = 0; x < U * 4; ++x) tl[x] = (ex[x] > 0.f) ? (st[x] - mc) * 1.44269504f : 0.f;
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const float w1 = (float)k / (float)(NC - 1), w0 = 1.f - w1;
            float acc = 0.f;
#pragma unroll
            for (int x = 0; x < U * 4; ++x)                // a term with p = 0 is 0 (tl is 0 there and the logarithm finite)
                acc += ex[x] * (tl[x] - __builtin_amdgcn_logf(fmaxf(fmaf(w1, q1[x], w0 * q0[x]), 1e-37f)));
            const double Ak = wave_sum((double)(acc * 0.693147181f));
            if (lane == 0) s_A[wave][k] = Ak;
        }
    } else if (drafts) {
        if (N > 0) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                float aj = 0.f;
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float p = ex[u * 4 + e];
                        if (p > 0.f) aj += p * (st[u * 4 + e] - f4get(dx[j][u], e) * invT);
                    }
                const double Aj = wave_sum((double)aj);
                if (lane == 0) s_A[wave][j] = Aj;
            }
        } else {
            auto sums = [&](auto load) {
                for (int j = 0; j < n; ++j) {
                    float aj = 0.f;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const float4 y = load(qbase + (size_t)j * V, u);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float p = ex[u * 4 + e];
                            if (p > 0.f) aj += p * (st[u * 4 + e] - f4get(y, e) * invT);
                        }
                    }
                    const double Aj = wave_sum((double)aj);
                    if (lane == 0) s_A[wave][j] = Aj;
                }
            };
            if (inside) sums([&](const float* row, int u) { return load_group(row, v(u)); });
            else with_row_loads(V, [&](auto load) { sums([&](const float* row, int u) { return load(row, at(u)); }); });
        }
    }
    __syncthreads();
    double* rec = a.stats + (((size_t)b * (gamma + 1) + i) * a.C3 + c) * a.RS;
    if (tid == 0) {
        ArgMax t = s_am[0];
        for (int w = 1; w < kWavesPerBlock; ++w) t = argmax_merge(t, s_am[w]);
        rec[0] = (double)mc;
        rec[1] = (s_redd[0] + s_redd[1]) + (s_redd[2] + s_redd[3]);
        rec[2] = (double)t.v;
        rec[3] = (double)t.i;
    }
    if (grid) {
        if (tid < TABED_GRID_CANDIDATES) {
            const double Zc = (s_redd[0] + s_redd[1]) + (s_redd[2] + s_redd[3]);
            // a chunk whose target logits are all -inf (masked) has no term in the sum: m_c Z_c would be -inf * 0 there
            rec[kStatHdr + tid] = ((s_A[0][tid] + s_A[1][tid]) + (s_A[2][tid] + s_A[3][tid])) + (Zc != 0.0 ? (double)mc * Zc : 0.0);
        }
    } else if (drafts && tid < n) {
        rec[kStatHdr + tid] = (s_A[0][tid] + s_A[1][tid]) + (s_A[2][tid] + s_A[3][tid]);
    }
}

template <int U, int N>
__global__ __launch_bounds__(kBlock) void k_stats(StatsArgs a) {
    stats_chunk<U, N>(a, blockIdx.x, blockIdx.y, blockIdx.z);
}

// =====================================================================================================
// Distances that do not ride in the records of k_stats: total variation and hard labels, also of the two-draft grid policy's
// candidate mixtures.  A workgroup sums, over its 4096-wide chunk of position i < gamma of sequence b,
//   MODE 0: |p - q_j|                         per draft j                (TVD, DW = n)
//   MODE 2: |p - mix_c|                       per candidate c            (TVD of the mixtures, n = 2)
//   MODE 3: arg-max_v q_j(v)                  per draft j                (hard labels; needs no target row)
//   MODE 4: arg-max_v mix_c(v)                per candidate c            (hard labels, n = 2)
// with mix_c = (1 - c/10) q_1 + (c/10) q_2.  Chunk sums go to dist[b][i][c][chunk][0]; chunk arg-maxes go to
// dist[b][i][c][chunk][0..1] as ((value, runner-up value) as two floats, index), lowest index on ties.
// |p - q| cannot be accumulated before the target row's normaliser is known: every workgroup of modes 0 and 2 first combines the
// row's records from k_stats (lse_p).  None of them needs anything of the accept chain, nor that anything of theirs, so that modes 0
// and 2 share k_finish's launch and modes 3 and 4 that of k_stats, and no launch of their own stands between the two.
// Whole verifications in us, with such a launch / now: total variation, V = 32000, 4 drafts, one sequence 21.1 / 17.1, V = 152064, 8
// sequences 66.9 / 52.2, V = 20000, 6 drafts, 9 sequences 34.5 / 22.8, V = 128256, 8 drafts, 32 sequences 149 / 141; mixtures of
// V = 100003, 24 sequences 64.1 / 56.4; hard labels, V = 32000, one sequence 24.1 / 20.8, V = 152064, 8 sequences 68.8 / 63.3.
// =====================================================================================================
struct DistArgs {
    int V, n, B, gamma, C3, RS, DW, Cd;
    const float* target;
    const float* dlogits;
    const double* dlse;
    const float* temperature;
    const double* stats;
    double* dist;
};

template <int MODE, int N>
__device__ __forceinline__ void dist_chunk(const DistArgs& a, int c, int i, int b) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int V = a.V, n = (N > 0) ? N : a.n, gamma = a.gamma;
    constexpr int NC = TABED_GRID_CANDIDATES;
    __shared__ double s_lse;
    __shared__ float s_hi[TABED_MAX_N], s_oml[TABED_MAX_N];
    __shared__ double s_sum[kWavesPerBlock][TABED_MAX_N];
    __shared__ ArgMax s_amx[kWavesPerBlock][TABED_MAX_N];
    __shared__ float s_sec[kWavesPerBlock][TABED_MAX_N];      // runner-up value beside every arg-max (mixtures only)

    const float* trow = a.target + ((size_t)b * (gamma + 1) + i) * V;
    const float* qbase = a.dlogits + (((size_t)i * a.B + b) * n) * V;
    const int cb = c * kChunkV;
    const bool inside = cb + kChunkV <= V;
    auto v = [&](int u) { return cb + (u * kBlock + tid) * 4; };
    auto at = [&](int u) { return group_at(v(u), V); };
    if (MODE >= 3) {
        // ---- hard labels: arg-max of every candidate distribution over this chunk
        const float T3 = a.temperature[b];
        const float invT3 = (T3 > 0.f) ? 1.f / T3 : 1.f;
        if (MODE == 3) {
            for (int j = 0; j < n; ++j) {                  // softmax is monotone: the arg-max of the raw logits
                ArgMax am{-INFINITY, 0x7fffffff};
                float4 y[4];
                with_row_loads(V, [&](auto load) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) y[u] = load(qbase + (size_t)j * V, at(u));
                });
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (at(u) + e >= v(u) && at(u) + e < V) am = argmax_merge(am, ArgMax{f4get(y[u], e), at(u) + e});
                am = wave_argmax(am);
                // fp32 logits compare exactly on both sides of any check: no runner-up is needed for these
                if (lane == 0) { s_amx[wave][j] = am; s_sec[wave][j] = -INFINITY; }
            }
        } else {
            if (tid < 2) {
                const double l = a.dlse[((size_t)i * a.B + b) * n + tid];
                const float hi = (float)l;
                s_hi[tid] = hi;
                s_oml[tid] = (float)(1.0 - (l - (double)hi));
            }
            float4 y0[4], y1[4];
            with_row_loads(V, [&](auto load) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    y0[u] = load(qbase, at(u));
                    y1[u] = load(qbase + (size_t)V, at(u));
                }
            });
            __syncthreads();
            float q0[16], q1[16];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float a0 = f4get(y0[u], e), a1 = f4get(y1[u], e);
                    q0[u * 4 + e] = (a0 > -INFINITY) ? __expf(a0 * invT3 - s_hi[0]) * s_oml[0] : 0.f;
                    q1[u * 4 + e] = (a1 > -INFINITY) ? __expf(a1 * invT3 - s_hi[1]) * s_oml[1] : 0.f;
                }
            for (int k = 0; k < NC; ++k) {
                const float w1 = (float)k / (float)(NC - 1), w0 = 1.f - w1;
                // the mixture is evaluated in fp32 here, a 64-bit evaluation can differ: the runner-up travels with the
                // arg-max so that a near-tie can be flagged where the label is known
                ArgMax am{-INFINITY, 0x7fffffff};
                float sec = -INFINITY;
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const int ve = at(x >> 2) + (x & 3);
                    if (ve >= v(x >> 2) && ve < V) {
                        const ArgMax cand{w0 * q0[x] + w1 * q1[x], ve};
                        const ArgMax win = argmax_merge(am, cand);
                        sec = fmaxf(sec, win.i == cand.i ? am.v : cand.v);      // the loser's value
                        am = win;
                    }
                }
                const ArgMax wam = wave_argmax(am);
                const float wsec = wave_max((am.i == wam.i) ? sec : am.v);
                if (lane == 0) { s_amx[wave][k] = wam; s_sec[wave][k] = wsec; }
            }
        }
        __syncthreads();
        if (tid < a.DW) {
            ArgMax t = s_amx[0][tid];
            float sec = s_sec[0][tid];
            for (int w = 1; w < kWavesPerBlock; ++w) {
                const ArgMax o = s_amx[w][tid];
                const ArgMax win = argmax_merge(t, o);
                sec = fmaxf(fmaxf(sec, s_sec[w][tid]), (win.i == o.i && o.i != t.i) ? t.v : o.v);
                t = win;
            }
            double* rec = a.dist + ((((size_t)b * gamma + i) * a.DW + tid) * a.Cd + c) * 2;
            rec[0] = __builtin_bit_cast(double, make_float2(t.v, sec));       // (arg-max value, runner-up value)
            rec[1] = (double)t.i;
        }
        return;
    }
    float4 tx[4];
    constexpr int NQ = (MODE != 0) ? 2 : N;
    float4 yq[NQ > 0 ? NQ : 1][4];                     // the draft rows, where they are requested up front
    with_row_loads(V, [&](auto load) {
#pragma unroll
        for (int u = 0; u < 4; ++u) tx[u] = load(trow, at(u));
#pragma unroll
        for (int j = 0; j < NQ; ++j)
#pragma unroll
            for (int u = 0; u < 4; ++u) yq[j][u] = load(qbase + (size_t)j * V, at(u));
    });
    if (!inside) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            mask_group(tx[u], at(u), v(u));
#pragma unroll
            for (int j = 0; j < NQ; ++j) mask_group(yq[j][u], at(u), v(u));
        }
    }
    const float T = a.temperature[b];
    const float invT = (T > 0.f) ? 1.f / T : 1.f;
    if (tid < n) {
        const double l = a.dlse[((size_t)i * a.B + b) * n + tid];
        const float hi = (float)l;
        s_hi[tid] = hi;
        s_oml[tid] = (float)(1.0 - (l - (double)hi));
    }
    if (wave == 0) {                                   // lse of target row (b, i) from its records
        const double* r0 = a.stats + ((size_t)b * (gamma + 1) + i) * a.C3 * a.RS;
        double m = -INFINITY, m0 = -INFINITY, z0 = 0.0;
        if (lane < a.C3) { m0 = r0[(size_t)lane * a.RS]; z0 = r0[(size_t)lane * a.RS + 1]; }      // (one trip for up to 64 chunks)
        m = m0;
        for (int cc = lane + kWave; cc < a.C3; cc += kWave) m = fmax(m, r0[(size_t)cc * a.RS]);
        m = wave_max(m);
        double Z = (m0 > -INFINITY) ? z0 * exp(m0 - m) : 0.0;
        for (int cc = lane + kWave; cc < a.C3; cc += kWave) {
            const double* r = r0 + (size_t)cc * a.RS;
            if (r[0] > -INFINITY) Z += r[1] * exp(r[0] - m);
        }
        Z = wave_sum(Z);
        if (lane == 0) s_lse = m + log(Z);
    }
    __syncthreads();
    const double lse = s_lse;
    const float lhi = (float)lse, loml = (float)(1.0 - (lse - (double)lhi));

    float pv[16];                                      // p of this thread's 16 elements
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float xe = f4get(tx[u], e);
            const float st = xe * invT;
            const bool ok = xe > -INFINITY;
            pv[u * 4 + e] = ok ? __expf(st - lhi) * loml : 0.f;
        }

    if (MODE == 0) {
        auto row = [&](int j, const float4 (&y)[4]) {
            float acc = 0.f;
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float ye = f4get(y[u], e);
                    const float q = (ye > -INFINITY) ? __expf(ye * invT - s_hi[j]) * s_oml[j] : 0.f;
                    acc += fabsf(pv[u * 4 + e] - q);
                }
            const double t = wave_sum((double)acc);
            if (lane == 0) s_sum[wave][j] = t;
        };
        if (N > 0) {
#pragma unroll
            for (int j = 0; j < N; ++j) row(j, yq[j]);
        } else {
            // two rows at a time: the next one is on its way while one is summed (past the last draft it is re-read)
            with_row_loads(V, [&](auto load) {
                float4 y[2][4];
                auto request = [&](int j, int set) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) y[set][u] = load(qbase + (size_t)min(j, n - 1) * V, at(u));
                };
                auto use = [&](int j, int set) {
                    if (!inside) {
#pragma unroll
                        for (int u = 0; u < 4; ++u) mask_group(y[set][u], at(u), v(u));
                    }
                    row(j, y[set]);
                };
                request(0, 0);
                for (int j = 0; j < n; j += 2) {
                    request(j + 1, 1);
                    use(j, 0);
                    request(j + 2, 0);
                    if (j + 1 < n) use(j + 1, 1);
                }
            });
        }
    } else {
        // both drafts' probabilities of this thread's 16 elements, then one candidate mixture at a time
        float q0[16], q1[16];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a0 = f4get(yq[0][u], e), a1 = f4get(yq[1][u], e);
                q0[u * 4 + e] = (a0 > -INFINITY) ? __expf(a0 * invT - s_hi[0]) * s_oml[0] : 0.f;
                q1[u * 4 + e] = (a1 > -INFINITY) ? __expf(a1 * invT - s_hi[1]) * s_oml[1] : 0.f;
            }
        for (int k = 0; k < NC; ++k) {
            const float w1 = (float)k / (float)(NC - 1), w0 = 1.f - w1;
            float acc = 0.f;
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const float mix = w0 * q0[x] + w1 * q1[x];
                acc += fabsf(pv[x] - mix);
            }
            const double t = wave_sum((double)acc);
            if (lane == 0) s_sum[wave][k] = t;
        }
    }
    __syncthreads();
    if (tid < a.DW)                                        // another workgroup of this launch adds the chunks
        publish_store(&a.dist[((((size_t)b * gamma + i) * a.DW + tid) * a.Cd + c) * 2],
                      (s_sum[0][tid] + s_sum[1][tid]) + (s_sum[2][tid] + s_sum[3][tid]));
}

// Target statistics and hard labels in one launch: the labels' workgroups first (nd of them), then k_stats'.
template <int U, int MODE>
__global__ __launch_bounds__(kBlock) void k_stats_labels(StatsArgs a, DistArgs d, int nd) {
    int g = blockIdx.y * gridDim.x + blockIdx.x;
    if (g < nd) {
        const int c = g % d.Cd, bi = g / d.Cd;
        dist_chunk<MODE, 0>(d, c, bi % d.gamma, bi / d.gamma);
    } else {
        g -= nd;
        const int c = g % a.C3, bi = g / a.C3;
        if (bi >= (a.gamma + 1) * a.B) return;             // (the last row of a grid of several)
        stats_chunk<U, 0>(a, c, bi % (a.gamma + 1), bi / (a.gamma + 1));
    }
}

static int pick_stats_unroll(const tabed_cfg& c, int nmax_u) {
    // Largest chunk that still gives the chip a few workgroups per compute unit.
    const long rows = (long)c.B * (c.gamma + 1);
    for (int U : {4, 2}) {
        if (U > nmax_u) continue;
        const long chunks = (c.V + kBlock * 4 * U - 1) / (kBlock * 4 * U);
        if (rows * chunks >= 1024) return U;           // measured on the serving shape: 1536 workgroups beat 768
    }
    return 1;
}

static int stats_chunks(const tabed_cfg& c, int U) { return (c.V + kBlock * 4 * U - 1) / (kBlock * 4 * U); }

// Grid of k_stats_labels.  A launch takes fewer than 2^32 threads a dimension, and four chunks a row of 65535 sequences with 32 positions
// are more: beyond 2^20 workgroups there is more than one row of them.  (k_finish with distances stays below: its workgroups reach
// 2^24 with eight chunks of 65535 x 32 positions, whose logits are 480 GB.)
static dim3 stats_labels_grid(const tabed_cfg& c, const WsLayout& L, int C3) {
    constexpr uint32_t kRow = 1u << 20;
    const uint32_t total = (uint32_t)(L.Cd * c.gamma + C3 * (c.gamma + 1)) * (uint32_t)c.B;
    return total <= kRow ? dim3(total) : dim3(kRow, (total + kRow - 1) / kRow);
}
dim3 stats_labels_grid(const tabed_cfg& c, const WsLayout& L) { return stats_labels_grid(c, L, stats_chunks(c, pick_stats_unroll(c, 4))); }

template <int N>
static void launch_stats_n(const ProfScope* prof, int U, dim3 grid, hipStream_t s, const StatsArgs& a) {
    if (U == 4) {
        if constexpr (N <= 4) launch(prof, k_stats<4, N>, grid, dim3(kBlock), 0, s, a);
    } else if (U == 2) {
        launch(prof, k_stats<2, N>, grid, dim3(kBlock), 0, s, a);
    } else {
        launch(prof, k_stats<1, N>, grid, dim3(kBlock), 0, s, a);
    }
}

// Draft counts that the passes over the vocabulary know at compile time (all rows of an element requested at once).
static int compiled_drafts(int n) { return (n <= 5 || n == 8) ? n : 0; }
#define TABED_FOR_DRAFTS(ncomp, CALL) \
    switch (ncomp) {                  \
        case 1: CALL(1); break;       \
        case 2: CALL(2); break;       \
        case 3: CALL(3); break;       \
        case 4: CALL(4); break;       \
        case 5: CALL(5); break;       \
        case 8: CALL(8); break;       \
        default: CALL(0); break;      \
    }

// =====================================================================================================
// Accept chain, distances, corrected / bonus token.
// Grid (chunk + 1, sequence b).  Every workgroup of a sequence first combines the chunk records of all
// gamma+1 target rows (fp64, fixed order), evaluates the gamma accept tests of Sec. 3 item 3 in parallel
// and takes k = the first failing position.  The last workgroup of the row (the "book-keeping" one) has
// no vocabulary chunk: it writes KL(p_i || q_i^(j)) and the bookkeeping outputs and, when asked to,
// advances the window and computes the next weights while its siblings work on the residual row.  For a
// sampling row the emitted token comes from f = max(0, p_k - q_k) (k < gamma) or f = p_gamma (k = gamma): every wave writes the mass of f over its 256-wide segments; the last
// workgroup of the sequence to arrive prefixes the segment masses in order, finds the segment the uniform
// falls into, and one wave re-evaluates that segment element by element.  A greedy row emits the arg-max of
// target row k and needs no vocabulary pass.
// =====================================================================================================
struct FinishArgs {
    int V, n, B, gamma, C3, RS, NSEG, C5, TS;
    uint64_t seed, round;
    const float* target;
    const float* dlogits;
    const double* dlse;
    const int32_t* dtok;
    const float* dq;
    const float* weights;
    const float* temperature;
    const float* u_acc;
    const float* u_res;
    const double* stats;
    const double* dist;   // [B][gamma][DW][Cd] chunk sums of dist_chunk, or nullptr (KL from the records)
    int DW, Cd;
    float dist_scale;     // 0.5 for total variation, 1 for KL
    int hard;             // 1: dist holds chunk arg-maxes and the distance is the token-mismatch indicator
    int hard_margin;      // 1: those arg-maxes are of fp32 mixtures: a near-tie flags the position
    int grid_kl;          // 1: the records of k_stats hold the KL sums of the DW candidate mixtures
    int fuse;             // 1: the call also advances every sequence's window and writes the next weights
    WindowArgs win;
    double* tstate;       // token tree: [B][kTsSlots] record of every sequence's walk, or nullptr (chain)
    float* wstage;        // [B][n] next weights, staged until every workgroup of the sequence has arrived
    double* seg;          // [B][2][NSEG]
    uint32_t* tickets;
    uint32_t* wtickets;   // [B] of the staged weights
    uint32_t* dtickets;   // [B] of the distances, where their workgroups are in this launch
    int early;            // 1: greedy rows' workgroups without book-keeping leave at once
    int32_t* accept_len;
    int32_t* out_tokens;
    float* dev;
    int32_t* n_valid;
    uint8_t* flags;
};

// exp(x - (hi + lo)), lo << 1.  The residual pass only locates a CDF crossing, whose margin (1e-6 of the
// total mass, flagged) is far above the ~1e-7 |x - hi| relative error of the fast exponential.
__device__ __forceinline__ float exp_shifted(float x, float hi, float one_minus_lo) {
    return __expf(x - hi) * one_minus_lo;
}

struct ResidRow {
    const float* trow;
    const float* qrows;   // n rows, stride V
    float invT, pmax, pinvZ;
    bool bonus;
};

// f, p and q for S groups of four consecutive elements, the groups that group_at gives for elements v[s] (v[s] % 4 == 0; f and p
// are 0 for elements before v[s] or past V; inside: no lane's group reaches past V).  Every load is issued before the first use; N is the compile-time number of drafts
// (0 = run time, the rows of four drafts at a time).
template <int N, int S>
__device__ __forceinline__ void resid_eval(const ResidRow& r, int n, int V, bool inside, const int (&v)[S], const float* s_hi,
                                           const float* s_lo, const float* s_w, float (&f)[S][4], float (&p)[S][4],
                                           float (&q)[S][4]) {
    float4 tx[S];
    float4 dx[(N > 0) ? N : 1][S];
    int at[S];
#pragma unroll
    for (int s = 0; s < S; ++s) at[s] = group_at(v[s], V);
    with_row_loads(V, [&](auto load) {
#pragma unroll
        for (int s = 0; s < S; ++s) tx[s] = load(r.trow, at[s]);
        if (N > 0 && !r.bonus) {
#pragma unroll
            for (int j = 0; j < N; ++j)
#pragma unroll
                for (int s = 0; s < S; ++s) dx[j][s] = load(r.qrows + (size_t)j * V, at[s]);
        }
    });
    if (!inside) {                                       // (f = max(0, p - q) is 0 with p, whatever q)
#pragma unroll
        for (int s = 0; s < S; ++s) mask_group(tx[s], at[s], v[s]);
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) q[s][e] = 0.f;
    if (!r.bonus) {
        if (N > 0) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const float w = s_w[j], hi = s_hi[j], lo = s_lo[j];
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float ye = f4get(dx[j][s], e);
                        if (ye > -INFINITY) q[s][e] += w * exp_shifted(ye * r.invT, hi, lo);
                    }
            }
        } else {
            constexpr int JB = 4;                          // draft rows requested together
            for (int j0 = 0; j0 < n; j0 += JB) {
                float4 y[JB][S];
                with_row_loads(V, [&](auto load) {
#pragma unroll
                    for (int jj = 0; jj < JB; ++jj)        // past the last draft: re-read, not used
#pragma unroll
                        for (int s = 0; s < S; ++s) y[jj][s] = load(r.qrows + (size_t)min(j0 + jj, n - 1) * V, at[s]);
                });
#pragma unroll
                for (int jj = 0; jj < JB; ++jj)
                    if (j0 + jj < n) {
                        const float w = s_w[j0 + jj], hi = s_hi[j0 + jj], lo = s_lo[j0 + jj];
#pragma unroll
                        for (int s = 0; s < S; ++s)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float ye = f4get(y[jj][s], e);
                                if (ye > -INFINITY) q[s][e] += w * exp_shifted(ye * r.invT, hi, lo);
                            }
                    }
            }
        }
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float xe = f4get(tx[s], e);
            const float pe = (xe > -INFINITY) ? __expf(xe * r.invT - r.pmax) * r.pinvZ : 0.f;
            p[s][e] = pe;
            f[s][e] = r.bonus ? pe : fmaxf(0.f, pe - q[s][e]);
        }
}

// Arg-max over the chunk arg-maxes of one (position, candidate): records are ((value, runner-up), index).
// *near: the runner-up over the whole row is within the margin of the winner.
__device__ __forceinline__ int hard_pred(const double* rec, int Cd, bool* near) {
    ArgMax am{-INFINITY, 0x7fffffff};
    float sec = -INFINITY;
    for (int cc = 0; cc < Cd; ++cc) {
        const float2 vs = __builtin_bit_cast(float2, rec[cc * 2]);
        const ArgMax o{vs.x, (int)rec[cc * 2 + 1]};
        const ArgMax win = argmax_merge(am, o);
        sec = fmaxf(fmaxf(sec, vs.y), (win.i == o.i && o.i != am.i) ? am.v : o.v);
        am = win;
    }
    *near = (am.v - sec) < kMargin * fabsf(am.v);
    return am.i;
}

// Segment masses of one thread's run [g0, g1) of the CDF, published by other workgroups: all of them requested together.
// A vocabulary of at most 262144 has 1024 segments, four per thread.
constexpr int kMaxSegRun = 4;
__device__ __forceinline__ void load_seg_run(const double* mass, int g0, int g1, double (&m)[kMaxSegRun]) {
#pragma unroll
    for (int q = 0; q < kMaxSegRun; ++q) m[q] = 0.0;
#pragma unroll
    for (int q = 0; q < kMaxSegRun; ++q)
        if (g0 + q < g1) m[q] = published_load(&mass[g0 + q]);
}
// The owner of the run that contains `target` walks it: first segment whose inclusive prefix exceeds the target, the last
// non-empty one if rounding lets none exceed it.
__device__ __forceinline__ void walk_seg_run(const double (&mR)[kMaxSegRun], const double (&mP)[kMaxSegRun], bool from_p, int g0,
                                             int g1, double excl, double target, int* s_seg, double* s_prefix) {
    double P = excl, Plast = excl;
    int gstar = -1, glast = g0;
#pragma unroll
    for (int q = 0; q < kMaxSegRun; ++q) {
        const double mg = from_p ? mP[q] : mR[q];
        if (g0 + q < g1 && gstar < 0) {
            if (mg > 0.0) { glast = g0 + q; Plast = P; }
            if (P + mg > target) gstar = g0 + q;
            else P += mg;
        }
    }
    if (gstar < 0) { gstar = glast; P = Plast; }
    *s_seg = gstar;
    *s_prefix = P;
}

// DK: whether the workgroups of the distances are in this launch.  0: no (KL, hard labels); 1, 2: total variation of the drafts, all
// rows of a chunk up front or one after the other; 3: of the two-draft grid's mixtures.  They come after all others in the
// grid, and the last to arrive of them and of the book-keeping workgroup, which knows how many positions count, adds a sequence's
// chunk sums and does what the book-keeping workgroup does otherwise: distances, window, next weights.
enum DistKind { kDistNone = 0, kDistUpFront = 1, kDistInTurn = 2, kDistMixtures = 3 };

template <int N, int DK>
__global__ __launch_bounds__(kBlock) void k_finish(FinishArgs a, DistArgs d) {
    extern __shared__ __attribute__((aligned(16))) double s_scale[];   // [gamma+1][C3]: exp(m_c - m_row)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int c = blockIdx.x, b = blockIdx.y;
    __shared__ double s_wpart[64], s_wx[TABED_MAX_N];    // window update (one wave)
    __shared__ int s_last;
    __shared__ float s_dev[DK != kDistNone ? TABED_MAX_GAMMA * TABED_MAX_N : 1];
    // the sum of a sequence's distances over their chunks, then window and next weights (all workgroups that it waits for are done)
    auto sum_distances = [&](bool greedy) {
        const int l8 = tid & 7, entries = a.gamma * a.DW;  // eight lanes an entry, each every eighth chunk in order
        for (int q0 = 0; q0 < entries; q0 += kBlock / 8) {
            const int q = q0 + (tid >> 3);
            const double* r0 = a.dist + ((size_t)b * entries + min(q, entries - 1)) * a.Cd * 2;
            double D = 0.0;
            for (int c0 = l8; c0 < a.Cd; c0 += 64) {
                double v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = published_load(&r0[min(c0 + 8 * u, a.Cd - 1) * 2]);
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (c0 + 8 * u < a.Cd) D += v[u];
            }
            D += dpp_f64<kDppXor1>(D);
            D += dpp_f64<kDppXor2>(D);
            D += dpp_f64<kDppHalfMirror>(D);
            const float e = (float)((double)a.dist_scale * D);
            if (l8 == 0 && q < entries) { a.dev[(size_t)b * entries + q] = e; s_dev[q] = e; }
        }
        if (!a.fuse) return;
        __syncthreads();
        if (tid >= kWave) return;
        const int nv = published_load(&a.n_valid[b]);
        WindowArgs wa = a.win;
        if (!greedy) wa.weights = a.wstage;                // (see the book-keeping workgroup below)
        window_update<true>(wa, b, lane, [&](int q) { return s_dev[q]; }, nv, s_wpart, s_wx);
        if (greedy) return;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        int second = 0;
        if (lane == 0) second = arrive(&a.wtickets[(size_t)b * a.TS], 2u) ? 1 : 0;
        if (__builtin_amdgcn_readfirstlane(second) && lane < a.n)
            a.win.weights[(size_t)b * a.n + lane] = published_load(&a.wstage[(size_t)b * a.n + lane]);
    };
    auto arrive_distances = [&]() -> bool {                // by all of a workgroup, its results published
        publish_barrier();
        if (tid == 0) s_last = arrive(&a.dtickets[(size_t)b * a.TS], (uint32_t)(a.Cd * a.gamma + 1)) ? 1 : 0;
        __syncthreads();
        return s_last != 0;
    };
    if constexpr (DK != kDistNone) {
        const int nf = (a.C5 + 1) * a.B;
        int g = blockIdx.x;
        if (g >= nf) {
            g -= nf;
            const int bi = g / a.Cd;
            b = bi / a.gamma;
            dist_chunk<DK == kDistMixtures ? 2 : 0, DK == kDistInTurn ? 0 : N>(d, g % a.Cd, bi % a.gamma, b);
            if (arrive_distances()) sum_distances(!(a.temperature[b] > 0.f));
            return;
        }
        b = g / (a.C5 + 1);
        c = g % (a.C5 + 1);
    }
    const int V = a.V, n = (N > 0) ? N : a.n, gamma = a.gamma, NSEG = a.NSEG, C3 = a.C3, RS = a.RS;

    __shared__ double s_rowm[TABED_MAX_GAMMA + 1], s_rowZ[TABED_MAX_GAMMA + 1], s_rowlse[TABED_MAX_GAMMA + 1];
    __shared__ int s_rowam[TABED_MAX_GAMMA + 1];
    __shared__ int s_ok[TABED_MAX_GAMMA];
    __shared__ uint32_t s_aflag[TABED_MAX_GAMMA + 1];
    __shared__ float s_hi[TABED_MAX_GAMMA][TABED_MAX_N], s_lo[TABED_MAX_GAMMA][TABED_MAX_N], s_w[TABED_MAX_N];
    __shared__ double s_redd[kWavesPerBlock];
    __shared__ int s_first[kWavesPerBlock], s_lastw[kWavesPerBlock], s_seg;
    __shared__ double s_prefix;
    __shared__ int s_y[TABED_MAX_GAMMA];                 // drafted tokens (hard labels)

    // ---- a greedy row has work for its book-keeping workgroup only.  Where workgroups queue for the chip the others leave at
    //      once (48 sequences of V = 152063, half of them greedy: 22.5 us, 27.5 if they read the records first); elsewhere waiting
    //      for the temperature before anything else is requested would be one more trip for everybody.
    const bool book = (c == a.C5);                        // the book-keeping workgroup of this sequence
    if (a.early && !book) {
        if (!(a.temperature[b] > 0.f)) return;
    }
    asm volatile("" ::: "memory");                         // (keeps that load in its branch)

    // ---- everything that does not depend on another load is requested first
    int y = -1;
    float rawy = 0.f, uacc = 0.f, qy = 0.f;
    if (tid < gamma) {
        y = a.dtok[(size_t)b * gamma + tid];
        uacc = a.u_acc ? a.u_acc[(size_t)b * gamma + tid] : tabed_uniform(a.seed, a.round, (uint32_t)b, (uint32_t)tid, 1);
        qy = a.dq[(size_t)b * gamma + tid];
        s_y[tid] = y;
    }
    for (int q = tid; q < gamma * n; q += kBlock) {      // draft log-sum-exps of every position, split hi + lo
        const double l = a.dlse[((size_t)(q / n) * a.B + b) * n + (q % n)];
        const float hi = (float)l;
        s_hi[q / n][q % n] = hi;
        s_lo[q / n][q % n] = (float)(1.0 - (l - (double)hi));      // 1 - lo, the first-order factor of exp(-lo)
    }
    if (tid < n) s_w[tid] = a.weights[(size_t)b * n + tid];
    const float T = a.temperature[b];

    // ---- combine the chunk records of every target row.  A row's C3 chunks sit in an aligned group of
    //      C3p lanes (C3p = power of two >= C3), so one wave combines 64 / C3p rows per pass with one
    //      load round trip; rows with more than 64 chunks fall back to one wave per row.
    const double* sb = a.stats + (size_t)b * (gamma + 1) * C3 * RS;
    if (C3 <= kWave) {
        int C3p = 1;
        while (C3p < C3) C3p <<= 1;
        const int rows_per_pass = kWave / C3p;
        const int cc = lane & (C3p - 1);
        for (int row0 = wave * rows_per_pass; row0 <= gamma; row0 += kWavesPerBlock * rows_per_pass) {
            const int row = row0 + lane / C3p;
            const bool live = (row <= gamma && cc < C3);
            double r0v = -INFINITY, r1v = 0.0;
            ArgMax am{-INFINITY, 0x7fffffff};
            if (live) {
                const double* r = sb + ((size_t)row * C3 + cc) * RS;
                r0v = r[0]; r1v = r[1];
                am = ArgMax{(float)r[2], (int)r[3]};
            }
            // all-reduce inside aligned groups of C3p lanes: DPP for the first four doublings (no LDS traffic),
            // ds_bpermute only beyond a 16-lane row
            double m = r0v;
            if (C3p > 1) m = fmax(m, dpp_f64<kDppXor1>(m));
            if (C3p > 2) m = fmax(m, dpp_f64<kDppXor2>(m));
            if (C3p > 4) m = fmax(m, dpp_f64<kDppHalfMirror>(m));
            if (C3p > 8) m = fmax(m, dpp_f64<kDppMirror>(m));
            for (int o = 16; o < C3p; o <<= 1) m = fmax(m, __shfl_xor(m, o));
            const double sc = (r0v > -INFINITY) ? exp(r0v - m) : 0.0;
            if (live) s_scale[row * C3 + cc] = sc;
            double Z = r1v * sc;
            if (C3p > 1) { Z += dpp_f64<kDppXor1>(Z); am = argmax_dpp_step<kDppXor1>(am); }
            if (C3p > 2) { Z += dpp_f64<kDppXor2>(Z); am = argmax_dpp_step<kDppXor2>(am); }
            if (C3p > 4) { Z += dpp_f64<kDppHalfMirror>(Z); am = argmax_dpp_step<kDppHalfMirror>(am); }
            if (C3p > 8) { Z += dpp_f64<kDppMirror>(Z); am = argmax_dpp_step<kDppMirror>(am); }
            for (int o = 16; o < C3p; o <<= 1) {
                Z += __shfl_xor(Z, o);
                const ArgMax other{__shfl_xor(am.v, o), __shfl_xor(am.i, o)};
                am = argmax_merge(am, other);
            }
            if (live && cc == 0) { s_rowm[row] = m; s_rowZ[row] = Z; s_rowlse[row] = m + log(Z); s_rowam[row] = am.i; }
        }
    } else {
        for (int row = wave; row <= gamma; row += kWavesPerBlock) {
            const double* r0 = sb + (size_t)row * C3 * RS;
            double m = -INFINITY;
            for (int cc = lane; cc < C3; cc += kWave) m = fmax(m, r0[(size_t)cc * RS]);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
            double Z = 0.0;
            ArgMax am{-INFINITY, 0x7fffffff};
            for (int cc = lane; cc < C3; cc += kWave) {
                const double* r = r0 + (size_t)cc * RS;
                const double sc = (r[0] > -INFINITY) ? exp(r[0] - m) : 0.0;
                s_scale[row * C3 + cc] = sc;
                Z += r[1] * sc;
                am = argmax_merge(am, ArgMax{(float)r[2], (int)r[3]});
            }
            Z = wave_sum(Z);
            am = wave_argmax(am);
            if (lane == 0) { s_rowm[row] = m; s_rowZ[row] = Z; s_rowlse[row] = m + log(Z); s_rowam[row] = am.i; }
        }
    }
    const bool greedy = !(T > 0.f);
    if (greedy && !book) return;
    const float invT = greedy ? 1.f : 1.f / T;
    const bool y_ok = (y >= 0 && y < V);
    if (tid < gamma && y_ok && !greedy) rawy = a.target[((size_t)b * (gamma + 1) + tid) * V + y];
    __syncthreads();

    // ---- gamma accept tests in parallel, k = first failure
    if (tid < gamma) {
        uint32_t flag = 0;
        bool ok;
        if (!y_ok) { ok = false; flag |= TABED_FLAG_DEGENERATE; }
        else if (greedy) ok = (y == s_rowam[tid]);
        else {
            const float py = (float)exp((double)(rawy * invT) - s_rowlse[tid]);
            const float lhs = uacc * qy;
            ok = lhs < py;
            if (fabs((double)lhs - (double)py) < (double)kMargin * fmax((double)lhs, (double)py))
                flag |= TABED_FLAG_ACCEPT_MARGIN;
        }
        s_ok[tid] = ok ? 1 : 0;
        s_aflag[tid] = flag;
    }
    if (tid == gamma) s_aflag[gamma] = 0;
    __syncthreads();
    int k = 0;
    while (k < gamma && s_ok[k]) ++k;
    const size_t out_idx = (size_t)b * (gamma + 1) + k;

    // ---- this workgroup's share of the residual (or bonus) row: 2 segments per wave, loads first
    ResidRow r;
    r.bonus = (k == gamma);
    r.invT = invT;
    r.trow = a.target + out_idx * V;
    r.pmax = (float)s_rowm[k];
    r.pinvZ = (float)(1.0 / s_rowZ[k]);
    r.qrows = r.bonus ? a.dlogits : a.dlogits + ((size_t)k * a.B + b) * n * V;
    const float* hi_k = s_hi[r.bonus ? 0 : k];
    const float* lo_k = s_lo[r.bonus ? 0 : k];
    constexpr int kSegPerChunk = kResidChunkV / kSegV;            // 8
    constexpr int kSegPerWave = kSegPerChunk / kWavesPerBlock;    // 2
    float f[kSegPerWave][4], p[kSegPerWave][4], qmix[kSegPerWave][4];
    int vs[kSegPerWave];
    if (!greedy && !book) {
#pragma unroll
        for (int s = 0; s < kSegPerWave; ++s) vs[s] = (c * kSegPerChunk + wave + s * kWavesPerBlock) * kSegV + lane * 4;
        resid_eval<N, kSegPerWave>(r, n, V, (c + 1) * kResidChunkV <= V, vs, hi_k, lo_k, s_w, f, p, qmix);
    }

    if (book) {
        if (DK != kDistNone) {
            // (distances: sum_distances)
        } else if (a.dist == nullptr) {
            // ---- distances: an entry per (position, draft or candidate mixture): its chunk sums times the scales
            //      computed above.  KL(p || q_j) = A_j / Z - lse_p + lse_j; a mixture's sums already hold its logarithm.
            //      Eight lanes add an entry's chunks, each every eighth one in order, eight requested at once; their sums are
            //      added in a fixed order (one thread per entry made this workgroup, which the window waits for, the last of
            //      its sequence: 11 us of a 20 us launch with 38 chunks).
            const int dw = a.grid_kl ? a.DW : n, l8 = tid & 7;
            for (int q0 = 0; q0 < gamma * dw; q0 += kBlock / 8) {
                const int q = q0 + (tid >> 3), qc = min(q, gamma * dw - 1), ii = qc / dw, j = qc % dw;
                const double* r0 = sb + (size_t)ii * C3 * RS + kStatHdr + j;
                const double lq = a.grid_kl ? 0.0 : a.dlse[((size_t)ii * a.B + b) * n + j];
                double A = 0.0;
                for (int c0 = l8; c0 < C3; c0 += 64) {
                    double v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = r0[(size_t)min(c0 + 8 * u, C3 - 1) * RS];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (c0 + 8 * u < C3) A += v[u] * s_scale[ii * C3 + c0 + 8 * u];
                }
                A += dpp_f64<kDppXor1>(A);
                A += dpp_f64<kDppXor2>(A);
                A += dpp_f64<kDppHalfMirror>(A);
                const double kl = A / s_rowZ[ii] - s_rowlse[ii] + lq;
                if (l8 == 0 && q < gamma * dw) publish_store(&a.dev[(size_t)b * gamma * dw + q], (float)kl);
            }
        } else {
            // ---- hard labels: 1 where a candidate's arg-max differs from the token emitted at the position.
            //      The label of the rejected position of a sampling row is the corrected token, which only
            //      the sampler's last workgroup knows: that entry is written there.
            for (int q = tid; q < gamma * a.DW; q += kBlock) {
                const int ii = q / a.DW;
                if (ii == k && !greedy) continue;
                const int label = ii < k ? s_y[ii] : (ii == k ? s_rowam[k] : -1);
                bool near;
                const int pred = hard_pred(a.dist + ((size_t)b * gamma * a.DW + q) * a.Cd * 2, a.Cd, &near);
                publish_store(&a.dev[(size_t)b * gamma * a.DW + q], pred == label ? 0.f : 1.f);
                if (near && a.hard_margin && ii <= k) atomicOr(&s_aflag[ii], (uint32_t)TABED_FLAG_SAMPLE_MARGIN);
            }
            __syncthreads();                               // (uniform: book and a.hard are) the flags are complete
        }
        if (tid <= gamma) {
            // accepted prefix, -1 padding, flags of the tests that were evaluated; slot k belongs to the sampler
            if (tid != k) {
                a.out_tokens[(size_t)b * (gamma + 1) + tid] = tid < k ? y : -1;
                a.flags[(size_t)b * (gamma + 1) + tid] = (uint8_t)(tid < k ? s_aflag[tid] : 0u);
            } else if (greedy) {
                a.out_tokens[out_idx] = s_rowam[k];
                a.flags[out_idx] = (uint8_t)s_aflag[k];
            }
        }
        if (tid == 0) {
            a.accept_len[b] = k;
            publish_store(&a.n_valid[b], k + 1 < gamma ? k + 1 : gamma);
            if (a.tstate != nullptr && greedy) {           // token tree: where the trunk stopped and what the target wants there
                double* ts = a.tstate + (size_t)b * kTsSlots;
                ts[kTsK] = (double)k;
                ts[kTsArgmax] = (double)s_rowam[k];
                ts[kTsZ1] = 0.0;
            }
        }
    }
    if constexpr (DK != kDistNone) {
        if (book) {
            if (arrive_distances()) sum_distances(greedy);
            return;
        }
    }
    const int nv_k = k + 1 < gamma ? k + 1 : gamma;
    auto dev_at = [&](int q) { return published_load(&a.dev[(size_t)b * gamma * a.win.dw + q]); };
    if (greedy) {
        // a greedy row is complete here: its single workgroup also advances the window when asked to
        if (a.fuse) {
            publish_barrier();                             // the distances above are acknowledged
            if (tid < kWave) window_update<true>(a.win, b, lane, dev_at, nv_k, s_wpart, s_wx);
        }
        return;
    }

    double* segR = a.seg + ((size_t)b * 2 + 0) * NSEG;
    double* segP = a.seg + ((size_t)b * 2 + 1) * NSEG;
    if (book) {
        // window + next weights, beside the sampler, which does not wait for them.  The weights are staged: the buffer
        // they go to may be the one the siblings are still reading this block's weights from.  Whoever comes second of
        // this workgroup and the sampler's last one, which knows that all siblings have read them, copies them out.
        // (With hard labels the window waits for the corrected token: there this workgroup is one of the siblings.)
        if (!a.hard) {
            if (!a.fuse) return;
            publish_barrier();                             // the distances above are acknowledged
            if (tid >= kWave) return;
            WindowArgs wa = a.win;
            wa.weights = a.wstage;
            window_update<true>(wa, b, lane, dev_at, nv_k, s_wpart, s_wx);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's staged weights are acknowledged
            int second = 0;
            if (lane == 0) second = arrive(&a.wtickets[(size_t)b * a.TS], 2u) ? 1 : 0;
            if (__builtin_amdgcn_readfirstlane(second) && lane < n)
                a.win.weights[(size_t)b * n + lane] = published_load(&a.wstage[(size_t)b * n + lane]);
            return;
        }
    } else {
#pragma unroll
        for (int s = 0; s < kSegPerWave; ++s) {
            const int seg = c * kSegPerChunk + wave + s * kWavesPerBlock;
            const double mf = (double)wave_sum((f[s][0] + f[s][1]) + (f[s][2] + f[s][3]));
            const double mp = (double)wave_sum((p[s][0] + p[s][1]) + (p[s][2] + p[s][3]));
            if (lane == 0 && seg < NSEG) { publish_store(&segR[seg], mf); publish_store(&segP[seg], mp); }
        }
    }
    publish_barrier();                                     // every wave's published stores are acknowledged
    if (tid == 0) s_last = arrive(&a.tickets[(size_t)b * a.TS], (uint32_t)(a.C5 + (a.hard ? 1 : 0))) ? 1 : 0;
    const float u_final = a.u_res ? a.u_res[b] : tabed_uniform(a.seed, a.round, (uint32_t)b, (uint32_t)gamma, 0);
    __syncthreads();
    if (!s_last) return;
    if (a.fuse && !a.hard && wave == kWavesPerBlock - 1) {  // every sibling has read this block's weights
        int second = 0;
        if (lane == 0) second = arrive(&a.wtickets[(size_t)b * a.TS], 2u) ? 1 : 0;
        if (__builtin_amdgcn_readfirstlane(second) && lane < n)
            a.win.weights[(size_t)b * n + lane] = published_load(&a.wstage[(size_t)b * n + lane]);
    }
    // hard labels: the rejected position's distances and the window update wait for the corrected token
    // returns the flag bit of a near-tie among the mixtures' arg-maxes at position k
    auto finish_hard = [&](int tok) -> uint32_t {          // wave 0 only
        bool any = false;
        if (k < gamma)
            for (int cidx = lane; cidx < a.DW; cidx += kWave) {
                bool near;
                const int pred = hard_pred(a.dist + (((size_t)b * gamma + k) * a.DW + cidx) * a.Cd * 2, a.Cd, &near);
                publish_store(&a.dev[((size_t)b * gamma + k) * a.DW + cidx], pred == tok ? 0.f : 1.f);
                any = any || near;
            }
        const uint32_t extra = (a.hard_margin && __ballot(any)) ? (uint32_t)TABED_FLAG_SAMPLE_MARGIN : 0u;
        if (a.fuse) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's published distances are acknowledged
            window_update<true>(a.win, b, lane, dev_at, nv_k, s_wpart, s_wx);
        }
        return extra;
    };

    // ---- last workgroup of sequence b: locate the segment, then the token
    const int S = (NSEG + kBlock - 1) / kBlock;            // at most kMaxSegRun consecutive segments per thread
    const int g0 = min(NSEG, tid * S), g1 = min(NSEG, g0 + S);
    uint32_t flag = s_aflag[k];
    double mR[kMaxSegRun], mP[kMaxSegRun];                 // requested together, kept for the walk below
    load_seg_run(segR, g0, g1, mR);
    load_seg_run(segP, g0, g1, mP);
    double runR = 0.0, runP = 0.0;
#pragma unroll
    for (int q = 0; q < kMaxSegRun; ++q) { runR += mR[q]; runP += mP[q]; }
    double run = runP, Z = 0.0, excl = 0.0, Z1 = 0.0;
    bool from_p = true;
    if (!r.bonus) {
        excl = block_exclusive_scan(runR, s_redd, &Z);
        if (Z > 0.0) { run = runR; from_p = false; Z1 = Z; }
        else { r.bonus = true; flag |= TABED_FLAG_DEGENERATE; }   // empty residual: draw from p_k
    }
    if (from_p) excl = block_exclusive_scan(runP, s_redd, &Z);
    if (a.tstate != nullptr && tid == 0) {                 // token tree: the first residual level is known here
        double* ts = a.tstate + (size_t)b * kTsSlots;
        ts[kTsK] = (double)k;
        ts[kTsRowMax] = s_rowm[k];
        ts[kTsRowZ] = s_rowZ[k];
        ts[kTsZ1] = Z1;                                    // 0: all gamma accepted, or an empty residual
        ts[kTsArgmax] = (double)s_rowam[k];
    }
    const double target = (double)u_final * Z;
    const int owner = block_find_owner(excl, run, target, s_first, s_lastw);
    if (owner < 0) {
        if (tid == 0) {
            a.out_tokens[out_idx] = 0;
            a.flags[out_idx] = (uint8_t)(flag | TABED_FLAG_SAMPLE_MARGIN | TABED_FLAG_DEGENERATE);
        }
        if (a.hard && tid < kWave) finish_hard(0);
        return;
    }
    if (tid == owner) walk_seg_run(mR, mP, from_p, g0, g1, excl, target, &s_seg, &s_prefix);
    __syncthreads();
    if (tid >= kWave) return;
    const int seg1 = __builtin_amdgcn_readfirstlane(s_seg), v1[1] = {seg1 * kSegV + lane * 4};
    float f1[1][4], p1[1][4], q1[1][4];
    resid_eval<N, 1>(r, n, V, (seg1 + 1) * kSegV <= V, v1, hi_k, lo_k, s_w, f1, p1, q1);
    const int v = group_at(v1[0], V);
    const double l1 = (double)f1[0][0], l2 = l1 + (double)f1[0][1], l3 = l2 + (double)f1[0][2], l4 = l3 + (double)f1[0][3];
    const double base = s_prefix + (wave_inclusive_scan(l4) - l4);
    const double cdf[4] = {base + l1, base + l2, base + l3, base + l4};
    int hit = -1, lastlive = -1;
#pragma unroll
    for (int e = 3; e >= 0; --e) {
        if (f1[0][e] > 0.f && cdf[e] > target) hit = e;
        if (lastlive < 0 && f1[0][e] > 0.f) lastlive = e;
    }
    const unsigned long long cross = __ballot(hit >= 0);
    const unsigned long long live = __ballot(lastlive >= 0);
    int pick;
    if (cross) pick = __ffsll((long long)cross) - 1;
    else if (live) { pick = 63 - __clzll((long long)live); flag |= TABED_FLAG_SAMPLE_MARGIN | TABED_FLAG_DEGENERATE; }
    else { pick = 0; flag |= TABED_FLAG_SAMPLE_MARGIN | TABED_FLAG_DEGENERATE; }
    if (a.hard) {
        const int e = cross ? hit : (live ? lastlive : 0);
        const int mine = (v + e < V) ? v + e : V - 1;
        flag |= finish_hard(__builtin_amdgcn_readlane(mine, pick));
    }
    if (lane == pick) {
        const int e = cross ? hit : (live ? lastlive : 0);
        const int tok = v + e;
        const double tol = (double)kMargin * Z;
        const double fe = (double)(e == 0 ? f1[0][0] : e == 1 ? f1[0][1] : e == 2 ? f1[0][2] : f1[0][3]);
        const double hi_edge = e == 0 ? cdf[0] : e == 1 ? cdf[1] : e == 2 ? cdf[2] : cdf[3];
        if (fabs(hi_edge - target) < tol && tok + 1 < V) flag |= TABED_FLAG_SAMPLE_MARGIN;
        if (tok > 0 && fabs((hi_edge - fe) - target) < tol) flag |= TABED_FLAG_SAMPLE_MARGIN;
        a.out_tokens[out_idx] = tok < V ? tok : V - 1;
        a.flags[out_idx] = (uint8_t)flag;
    }
}

hipError_t launch_verify(const tabed_cfg& c, const WsLayout& L, char* ws, uint64_t round,
                         const float* target_logits, const float* draft_logits, const double* draft_lse,
                         const int32_t* draft_tokens, const float* draft_q, const float* weights,
                         const float* temperature, const float* u_acc, const float* u_res, int32_t* accept_len,
                         int32_t* out_tokens, float* dev, int32_t* n_valid, uint8_t* flags, float* ring,
                         int32_t* ring_head, int32_t* ring_count, float* next_weights, bool tree, hipStream_t s) {
    const bool grid_in_stats = (c.policy == 2 && c.distance == 0);   // the KL of the two-draft grid's mixtures rides in the statistics pass
    const bool second_pass = (c.distance != 0);                      // distances that the records of k_stats do not hold
    const bool labels = (c.distance == 2);
    const int ncomp = compiled_drafts(c.n);
    // the statistics pass: rows one after the other for three and five drafts, where all of them up front took more registers
    // than the trips saved are worth (12 sequences of V = 128256, us: 3 drafts 17.5 against 18.5, 5 drafts 24.0 against 26.0),
    // and where it reads no draft row
    const int scomp = (second_pass || ncomp == 3 || ncomp == 5) ? 0 : ncomp;
    const int U = pick_stats_unroll(c, scomp > 4 ? 2 : 4), C3 = stats_chunks(c, U);
    DistArgs d{};
    d.V = c.V; d.n = c.n; d.B = c.B; d.gamma = c.gamma; d.C3 = C3; d.RS = L.RS; d.DW = L.DW; d.Cd = L.Cd;
    d.target = target_logits; d.dlogits = draft_logits; d.dlse = draft_lse; d.temperature = temperature;
    d.dist = reinterpret_cast<double*>(ws + L.off_dist);
    {
        ProfScope prof(TABED_K_STATS, s, labels ? TABED_K_DIST : -1);
        StatsArgs a;
        a.V = c.V; a.n = c.n; a.B = c.B; a.gamma = c.gamma; a.RS = L.RS; a.C3 = C3;
        a.with_drafts = second_pass ? 0 : 1;
        a.grid = grid_in_stats ? 1 : 0;
        a.target = target_logits; a.dlogits = draft_logits; a.dlse = draft_lse; a.temperature = temperature;
        a.stats = reinterpret_cast<double*>(ws + L.off_stats);
        const dim3 grid(C3, c.gamma + 1, c.B);
        d.stats = a.stats;
        if (labels) {
            const int nd = L.Cd * c.gamma * c.B;
            const dim3 both = stats_labels_grid(c, L, C3);
#define TABED_LABELS(U_) (c.policy != 2 ? launch(&prof, k_stats_labels<U_, 3>, both, dim3(kBlock), 0, s, a, d, nd) \
                                        : launch(&prof, k_stats_labels<U_, 4>, both, dim3(kBlock), 0, s, a, d, nd))
            if (U == 1) TABED_LABELS(1);
            else if (U == 2) TABED_LABELS(2);
            else TABED_LABELS(4);
#undef TABED_LABELS
        } else
#define TABED_STATS(N_) launch_stats_n<N_>(&prof, U, grid, s, a)
        switch (scomp) {
            case 1: TABED_STATS(1); break;
            case 2: TABED_STATS(2); break;
            case 4: TABED_STATS(4); break;
            case 8: TABED_STATS(8); break;
            default: TABED_STATS(0); break;
        }
#undef TABED_STATS
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    ProfScope prof(TABED_K_RESID, s, second_pass && !labels ? TABED_K_DIST : -1);
    FinishArgs a;
    a.V = c.V; a.n = c.n; a.B = c.B; a.gamma = c.gamma; a.C3 = C3; a.RS = L.RS; a.NSEG = L.NSEG; a.C5 = L.C5; a.TS = L.TS;
    a.seed = c.seed; a.round = round;
    a.target = target_logits; a.dlogits = draft_logits; a.dlse = draft_lse; a.dtok = draft_tokens; a.dq = draft_q;
    a.weights = weights; a.temperature = temperature; a.u_acc = u_acc; a.u_res = u_res;
    a.stats = reinterpret_cast<const double*>(ws + L.off_stats);
    a.dist = second_pass ? reinterpret_cast<const double*>(ws + L.off_dist) : nullptr;
    a.DW = L.DW; a.Cd = L.Cd; a.dist_scale = (c.distance == 1) ? 0.5f : 1.f; a.hard = (c.distance == 2) ? 1 : 0;
    a.hard_margin = (c.distance == 2 && c.policy == 2) ? 1 : 0;
    a.grid_kl = grid_in_stats ? 1 : 0;
    a.fuse = (ring != nullptr) ? 1 : 0;
    a.win = window_args(c, round + 1, ring, ring_head, ring_count, next_weights);   // the weights of the NEXT round
    a.wstage = reinterpret_cast<float*>(ws + L.off_wstage);
    a.tstate = tree ? reinterpret_cast<double*>(ws + L.off_tstate) : nullptr;
    a.seg = reinterpret_cast<double*>(ws + L.off_seg);
    a.tickets = reinterpret_cast<uint32_t*>(ws + L.off_tickets) + 2 * (size_t)c.B * L.TS;
    a.wtickets = reinterpret_cast<uint32_t*>(ws + L.off_tickets) + 1 * (size_t)c.B * L.TS;
    a.accept_len = accept_len; a.out_tokens = out_tokens; a.dev = dev; a.n_valid = n_valid; a.flags = flags;
    a.dtickets = reinterpret_cast<uint32_t*>(ws + L.off_tickets) + 3 * (size_t)c.B * L.TS;
    const int finishers = (L.C5 + 1) * c.B;              // with the book-keeping workgroup of every sequence
    a.early = finishers > 1024 ? 1 : 0;
    const size_t lds = sizeof(double) * (size_t)(c.gamma + 1) * C3;
    if (second_pass && !labels) {
        // All draft rows of a chunk up front while the registers of that (16 a row) leave the whole grid resident at once, one row after
        // the other beyond, where they cost more workgroups than the trips saved are worth (V = 50261, 3 drafts, 12 sequences, 936 workgroups: 25.3 / 26.0 us;
        // as a launch of their own, 1536 workgroups of V = 32000 with 2, 4 and 8 drafts 17.7 / 11.9, 27.9 / 18.8, 58.6 / 33.9).  Eight drafts
        // beyond: k_finish without a compile-time draft count has 81 registers instead of 117 (V = 128256, 32 sequences 165 us, 182;
        // 141 with two rows at a time).  (The registers decide: with the records' scales, at most 17 KB, a workgroup has 26 KB of LDS, six
        // of which fit a compute unit.)
        const long nd = (long)L.Cd * c.gamma * c.B;
        const dim3 grid((unsigned)(finishers + nd));
        const bool up_front = finishers + nd <= 256 * (ncomp <= 4 ? 4 : ncomp == 5 ? 3 : 2);
#define TABED_FINISH(N_)                                                                                          \
    up_front ? launch(&prof, k_finish<N_, N_ != 0 ? kDistUpFront : kDistInTurn>, grid, dim3(kBlock), lds, s, a, d) \
             : launch(&prof, k_finish<N_ != 8 ? N_ : 0, kDistInTurn>, grid, dim3(kBlock), lds, s, a, d)
        if (c.policy == 2) launch(&prof, k_finish<2, kDistMixtures>, grid, dim3(kBlock), lds, s, a, d);
        else { TABED_FOR_DRAFTS(ncomp, TABED_FINISH) }
#undef TABED_FINISH
        return hipGetLastError();
    }
    const dim3 grid(L.C5 + 1, c.B);
#define TABED_FINISH(N_) launch(&prof, k_finish<N_, kDistNone>, grid, dim3(kBlock), lds, s, a, d)
    TABED_FOR_DRAFTS(ncomp, TABED_FINISH)
#undef TABED_FINISH
    return hipGetLastError();
}

// =====================================================================================================
// Token tree (Sec. 6.1, "Verification: Integrating Token Tree"): width sibling candidates per position, all
// from the position's ensembled distribution; candidate 0 is the trunk token the chain verifies, candidates
// 1..width-1 are leaves.  tabed_verify's kernels walk the trunk and leave, per sequence, where it stopped (k),
// the target row's normaliser there and the mass Z_1 of the first residual.  The passes below finish the walk
// at position k by multi-round rejection sampling: with f_0 = p_k, Z_0 = 1 and
//     f_c(v) = max(0, f_{c-1}(v) / Z_{c-1} - q_k(v)),   Z_c = sum_v f_c(v),
// sibling c is accepted iff u_c q_k(y_c) Z_c < f_c(y_c); an accepted sibling is emitted and followed by a
// bonus token from the target's distribution after it (its leaf row); if all are rejected the corrected
// token comes from f_width.  Sibling 1 needs no pass (Z_1 is known), level L >= 2 is one pass over the row, which either decides
// sibling L or (L = width) draws the corrected token, and the token after an accepted leaf is one pass over that leaf's row.
// A sequence needs at most width - 1 passes, one after the other, and is in one of them at a time: a launch does the next pass of every
// sequence, whichever it is, and the first one tests sibling 1 as well (every workgroup for itself).  Width 2 takes one launch, width 3
// two; sequences whose walk is over leave at once.  (With launches of their own for the test, each level and the bonus token, two more
// each: a round of V = 32000, 4 drafts, 4 sequences, width 3
// 152.8 us, now 142.9; width 2 with 16 sequences 165.0, 155.9.)
// =====================================================================================================
struct TreeArgs {
    int V, n, B, gamma, S, NSEG, C5, TS;   // S = width - 1 siblings per position
    uint64_t seed, round;
    const float* target;                   // [B,gamma+1,V]
    const float* leaf_logits;              // [B,gamma,S,V]
    const float* dlogits;                  // [gamma,B,n,V]
    const double* dlse;                    // [gamma,B,n]
    const int32_t* sib_tokens;             // [B,gamma,S]
    const float* sib_q;                    // [B,gamma,S]
    const float* weights;
    const float* temperature;
    const float* u_res;
    const float* u_acc_sib;                // [B,gamma,S] or nullptr
    double* tstate;                        // [B][kTsSlots]
    const double* segP;                    // [B][2][NSEG] of tabed_verify's residual pass: slot 1 = masses of p_k
    double* tseg;                          // [B][2][NSEG]
    uint32_t* tickets;                     // [B] of this pass
    int32_t* out_tokens;
    uint8_t* flags;
    int32_t* leaf;
    int32_t* n_out;
};

// f_L(y) / Z_L's numerator chain at one token, in fp64, on the interface value q(y):
// returns f_{L-1}(y) / Z_{L-1} (the minuend of level L) given p(y), q(y) and the masses of the lower levels.
__device__ __forceinline__ double tree_minuend(int L, double py, double qy, double Z1, double Z2) {
    double m = py;                                          // level 1: f_0 / Z_0 = p
    if (L >= 2) m = fmax(0.0, m - qy) / Z1;
    if (L >= 3) m = fmax(0.0, m - qy) / Z2;
    return m;
}

// Sibling L's accept test (Z = Z_L).  Returns true if accepted; *flag gets the margin bit.
__device__ __forceinline__ bool tree_test(int L, double py, double qy, double Z1, double Z2, double Z, float u, uint32_t* flag) {
    const double minuend = tree_minuend(L, py, qy, Z1, Z2);
    const double fy = fmax(0.0, minuend - qy), lhs = (double)u * qy * Z;
    if (fabs(lhs - fy) < (double)kMargin * fmax(minuend, qy)) *flag |= TABED_FLAG_ACCEPT_MARGIN;
    return lhs < fy;
}

struct TreeWalk {
    int status, index, k;                                   // kTree*; next level or accepted sibling; the rejected position
    uint32_t flag;                                          // flags of position k so far
};

// Where the walk of sequence b starts: sibling 1's test, or the greedy row's match.  All threads alike.
__device__ __forceinline__ TreeWalk tree_begin(const TreeArgs& a, int b) {
    const double* ts = a.tstate + (size_t)b * kTsSlots;
    const int gamma = a.gamma, S = a.S, V = a.V, k = __builtin_amdgcn_readfirstlane((int)ts[kTsK]);
    const float T = a.temperature[b];
    TreeWalk t{kTreeDone, 0, k, 0};
    if (k >= gamma || S == 0) return t;
    const size_t so = ((size_t)b * gamma + k) * S;
    if (!(T > 0.f)) {
        const int top = (int)ts[kTsArgmax];
        for (int sidx = 1; sidx <= S && t.status == kTreeDone; ++sidx)
            if (a.sib_tokens[so + sidx - 1] == top) { t.status = kTreeLeaf; t.index = sidx; }
    } else if (ts[kTsZ1] > 0.0) {
        // the chain's corrected token (drawn from level 1) is replaced: by a leaf, or by a draw from level width
        t.flag = a.flags[(size_t)b * (gamma + 1) + k] & ~(uint32_t)(TABED_FLAG_SAMPLE_MARGIN | TABED_FLAG_DEGENERATE);
        const int y = a.sib_tokens[so];
        t.status = kTreePending; t.index = 2;
        if (y >= 0 && y < V) {
            const double lse = ts[kTsRowMax] + log(ts[kTsRowZ]);
            const double py = exp((double)(a.target[((size_t)b * (gamma + 1) + k) * V + y] * (1.f / T)) - lse);
            const float u = a.u_acc_sib ? a.u_acc_sib[so]
                                        : tabed_uniform(a.seed, a.round, (uint32_t)b, (uint32_t)k + kSiblingStride, 1);
            if (tree_test(1, py, (double)a.sib_q[so], 0.0, 0.0, ts[kTsZ1], u, &t.flag)) { t.status = kTreeLeaf; t.index = 1; }
        } else {
            t.flag |= TABED_FLAG_DEGENERATE;
        }
    }
    t.status = __builtin_amdgcn_readfirstlane(t.status);
    t.index = __builtin_amdgcn_readfirstlane(t.index);
    return t;
}

// Locates, in the workgroup that finishes a sequence, the 256-wide segment whose prefix of masses crosses
// target = u * Z; thread `tid` owns segments [g0, g1).  Returns false if every mass is zero.
__device__ __forceinline__ bool tree_pick_segment(const double* mass, int g0, int g1, double excl, double run, double target,
                                                  int* s_first, int* s_lastw, int* s_seg, double* s_prefix) {
    const int owner = block_find_owner(excl, run, target, s_first, s_lastw);
    if (owner < 0) return false;
    if ((int)threadIdx.x == owner) {
        double P = excl, Plast = excl;
        int gstar = -1, glast = g0;
        for (int g = g0; g < g1; ++g) {
            const double mg = published_load(&mass[g]);
            if (mg > 0.0) { glast = g; Plast = P; }
            if (P + mg > target) { gstar = g; break; }
            P += mg;
        }
        if (gstar < 0) { gstar = glast; P = Plast; }
        *s_seg = gstar;
        *s_prefix = P;
    }
    __syncthreads();
    return true;
}

// One wave: given the four values of every lane's group inside the chosen segment, the token where the prefix
// crosses target, with the margin flags of the sampler.  Returns the token on every lane.
__device__ __forceinline__ int tree_pick_token(const float (&f)[4], int v, int V, double prefix, double target, double Z,
                                               uint32_t* flag) {
    const int lane = threadIdx.x & 63;
    const double l1 = (double)f[0], l2 = l1 + (double)f[1], l3 = l2 + (double)f[2], l4 = l3 + (double)f[3];
    const double base = prefix + (wave_inclusive_scan(l4) - l4);
    const double cdf[4] = {base + l1, base + l2, base + l3, base + l4};
    int hit = -1, lastlive = -1;
#pragma unroll
    for (int e = 3; e >= 0; --e) {
        if (f[e] > 0.f && cdf[e] > target) hit = e;
        if (lastlive < 0 && f[e] > 0.f) lastlive = e;
    }
    const unsigned long long cross = __ballot(hit >= 0);
    const unsigned long long live = __ballot(lastlive >= 0);
    int pick;
    if (cross) pick = __ffsll((long long)cross) - 1;
    else if (live) { pick = 63 - __clzll((long long)live); *flag |= TABED_FLAG_SAMPLE_MARGIN | TABED_FLAG_DEGENERATE; }
    else { pick = 0; *flag |= TABED_FLAG_SAMPLE_MARGIN | TABED_FLAG_DEGENERATE; }
    const int e = cross ? hit : (live ? lastlive : 0);
    int tok = v + e;
    uint32_t mine = 0;
    if (lane == pick) {
        const double tol = (double)kMargin * Z;
        double fe = 0.0, hi_edge = 0.0;
#pragma unroll
        for (int x = 0; x < 4; ++x)                        // (not f[e]: the arrays stay in registers)
            if (x == e) { fe = (double)f[x]; hi_edge = cdf[x]; }
        if (fabs(hi_edge - target) < tol && tok + 1 < V) mine |= TABED_FLAG_SAMPLE_MARGIN;
        if (tok > 0 && fabs((hi_edge - fe) - target) < tol) mine |= TABED_FLAG_SAMPLE_MARGIN;
    }
    tok = tok < V ? tok : V - 1;
    *flag |= (uint32_t)__builtin_amdgcn_readlane((int)mine, pick);
    return __builtin_amdgcn_readlane(tok, pick);
}

// Level L = w.index of a pending sequence (one of its C5 workgroups).
template <int N>
__device__ __forceinline__ void tree_level(const TreeArgs& a, int c, int b, const TreeWalk& w) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, L = w.index, k = w.k;
    double* ts = a.tstate + (size_t)b * kTsSlots;
    const int V = a.V, n = (N > 0) ? N : a.n, gamma = a.gamma, S = a.S, NSEG = a.NSEG;
    const float T = a.temperature[b];
    const double Z1 = ts[kTsZ1], Z2 = ts[kTsZ2];
    const float invZ1 = (float)(1.0 / Z1), invZ2 = (L >= 3) ? (float)(1.0 / Z2) : 0.f;

    __shared__ float s_hi[TABED_MAX_N], s_lo[TABED_MAX_N], s_w[TABED_MAX_N];
    __shared__ double s_redd[kWavesPerBlock];
    __shared__ int s_last, s_first[kWavesPerBlock], s_lastw[kWavesPerBlock], s_seg;
    __shared__ double s_prefix;
    if (tid < n) {
        const double l = a.dlse[((size_t)k * a.B + b) * n + tid];
        const float hi = (float)l;
        s_hi[tid] = hi;
        s_lo[tid] = (float)(1.0 - (l - (double)hi));
        s_w[tid] = a.weights[(size_t)b * n + tid];
    }
    __syncthreads();
    ResidRow r;
    r.bonus = false;
    r.invT = 1.f / T;
    r.trow = a.target + ((size_t)b * (gamma + 1) + k) * V;
    r.pmax = (float)ts[kTsRowMax];
    r.pinvZ = (float)(1.0 / ts[kTsRowZ]);
    r.qrows = a.dlogits + ((size_t)k * a.B + b) * n * V;
    // level L from the elementwise values: f_1 = max(0, p - q), f_2 = max(0, f_1 / Z_1 - q), f_3 = max(0, f_2 / Z_2 - q)
    auto level = [&](float f1, float q) {
        float f = fmaxf(0.f, f1 * invZ1 - q);
        if (L >= 3) f = fmaxf(0.f, f * invZ2 - q);
        return f;
    };
    constexpr int kSegPerChunk = kResidChunkV / kSegV, kSegPerWave = kSegPerChunk / kWavesPerBlock;
    {
        float f[kSegPerWave][4], p[kSegPerWave][4], q[kSegPerWave][4];
        int vs[kSegPerWave];
#pragma unroll
        for (int sg = 0; sg < kSegPerWave; ++sg) vs[sg] = (c * kSegPerChunk + wave + sg * kWavesPerBlock) * kSegV + lane * 4;
        resid_eval<N, kSegPerWave>(r, n, V, (c + 1) * kResidChunkV <= V, vs, s_hi, s_lo, s_w, f, p, q);
#pragma unroll
        for (int sg = 0; sg < kSegPerWave; ++sg) {
            const int seg = c * kSegPerChunk + wave + sg * kWavesPerBlock;
            float acc = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc += level(f[sg][e], q[sg][e]);
            const double m = (double)wave_sum(acc);
            if (lane == 0 && seg < NSEG) publish_store(&a.tseg[((size_t)b * 2 + 0) * NSEG + seg], m);
        }
    }
    publish_barrier();
    if (tid == 0) s_last = arrive(&a.tickets[(size_t)b * a.TS], (uint32_t)a.C5) ? 1 : 0;
    __syncthreads();
    if (!s_last) return;

    // ---- last workgroup of the sequence: the level's mass, then sibling L's test or the corrected token
    const double* massL = a.tseg + ((size_t)b * 2 + 0) * NSEG;
    const double* massP = a.segP + ((size_t)b * 2 + 1) * NSEG;
    const int SPT = (NSEG + kBlock - 1) / kBlock;
    const int g0 = min(NSEG, tid * SPT), g1 = min(NSEG, g0 + SPT);
    if (tid == 0) { a.leaf[b] = 0; a.n_out[b] = k + 1; }    // (unless a leaf is accepted after all)
    double run = 0.0;
    for (int g = g0; g < g1; ++g) run += published_load(&massL[g]);
    double Z;
    double excl = block_exclusive_scan(run, s_redd, &Z);
    const size_t fidx = (size_t)b * (gamma + 1) + k;
    uint32_t flag = w.flag;
    const bool degenerate = !(Z > 0.0);
    const double* mass = massL;
    if (degenerate) {
        // empty residual (the lower level equals q): the token is drawn from p_k, whose segment masses the
        // chain's residual pass left behind
        flag |= TABED_FLAG_DEGENERATE;
        run = 0.0;
        for (int g = g0; g < g1; ++g) run += massP[g];
        excl = block_exclusive_scan(run, s_redd, &Z);
        mass = massP;
        r.bonus = true;
    } else if (L <= S) {
        if (tid == 0) {
            const size_t so = ((size_t)b * gamma + k) * S + (L - 1);
            const int y = a.sib_tokens[so];
            int decided = 0;
            if (y >= 0 && y < V) {
                const double lse = ts[kTsRowMax] + log(ts[kTsRowZ]);
                const double py = exp((double)(r.trow[y] * r.invT) - lse);
                const float u = a.u_acc_sib ? a.u_acc_sib[so]
                                            : tabed_uniform(a.seed, a.round, (uint32_t)b, (uint32_t)k + (uint32_t)L * kSiblingStride, 1);
                if (tree_test(L, py, (double)a.sib_q[so], Z1, Z2, Z, u, &flag)) decided = 1;
            } else {
                flag |= TABED_FLAG_DEGENERATE;
            }
            a.flags[fidx] = (uint8_t)flag;
            if (decided) { ts[kTsStatus] = (double)kTreeLeaf; ts[kTsIndex] = (double)L; }
            else { ts[kTsStatus] = (double)kTreePending; ts[kTsIndex] = (double)(L + 1); ts[kTsZ2] = Z; }   // L = 2: widths above 3 would need a Z_3
        }
        return;                                            // the next pass continues (or the leaf's bonus pass)
    }
    const float u = a.u_res ? a.u_res[b] : tabed_uniform(a.seed, a.round, (uint32_t)b, (uint32_t)gamma, 0);
    const double target = (double)u * Z;
    if (!tree_pick_segment(mass, g0, g1, excl, run, target, s_first, s_lastw, &s_seg, &s_prefix)) {
        if (tid == 0) {
            a.out_tokens[fidx] = 0;
            a.flags[fidx] = (uint8_t)(flag | TABED_FLAG_SAMPLE_MARGIN | TABED_FLAG_DEGENERATE);
            ts[kTsStatus] = (double)kTreeDone;
        }
        return;
    }
    if (tid >= kWave) return;
    const int seg1 = __builtin_amdgcn_readfirstlane(s_seg), v1[1] = {seg1 * kSegV + lane * 4};
    float f1[1][4], p1[1][4], q1[1][4], fl[4];
    resid_eval<N, 1>(r, n, V, (seg1 + 1) * kSegV <= V, v1, s_hi, s_lo, s_w, f1, p1, q1);
#pragma unroll
    for (int e = 0; e < 4; ++e) fl[e] = degenerate ? p1[0][e] : level(f1[0][e], q1[0][e]);
    const int tok = tree_pick_token(fl, group_at(v1[0], V), V, s_prefix, target, Z, &flag);
    if (lane == 0) {
        a.out_tokens[fidx] = tok;
        a.flags[fidx] = (uint8_t)flag;
        ts[kTsStatus] = (double)kTreeDone;
    }
}

// Bonus token after an accepted leaf: a draw from softmax(leaf row / T) with the round's u_res (arg-max for a
// greedy row).  Every wave leaves, per 256-wide segment, the maximum of the scaled logits and the sum of
// exp(. - that maximum); the last workgroup combines them (fp64, segment order), finds the segment the uniform
// falls into and re-evaluates it.  Greedy: per-segment (value, index) arg-max records, merged lowest index first.
__device__ __forceinline__ void tree_bonus(const TreeArgs& a, int c, int b, const TreeWalk& w) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double* ts = a.tstate + (size_t)b * kTsSlots;
    const int V = a.V, gamma = a.gamma, S = a.S, NSEG = a.NSEG;
    const int k = w.k, sidx = w.index;
    const float T = a.temperature[b];
    const bool greedy = !(T > 0.f);
    const float invT = greedy ? 1.f : 1.f / T;
    const size_t so = ((size_t)b * gamma + k) * S + (sidx - 1);
    const float* row = a.leaf_logits + so * V;
    double* rec0 = a.tseg + ((size_t)b * 2 + 0) * NSEG;    // sampling: segment sum;  greedy: arg-max value
    double* rec1 = a.tseg + ((size_t)b * 2 + 1) * NSEG;    // sampling: segment max;  greedy: arg-max index

    __shared__ double s_redd[kWavesPerBlock];
    __shared__ float s_redf[kWavesPerBlock];
    __shared__ ArgMax s_am[kWavesPerBlock];
    __shared__ int s_last, s_first[kWavesPerBlock], s_lastw[kWavesPerBlock], s_seg;
    __shared__ double s_prefix;

    constexpr int kSegPerChunk = kResidChunkV / kSegV, kSegPerWave = kSegPerChunk / kWavesPerBlock;
    float4 x[kSegPerWave];
    int v[kSegPerWave], at[kSegPerWave];
#pragma unroll
    for (int sg = 0; sg < kSegPerWave; ++sg) {
        v[sg] = (c * kSegPerChunk + wave + sg * kWavesPerBlock) * kSegV + lane * 4;
        at[sg] = group_at(v[sg], V);
    }
    with_row_loads(V, [&](auto load) {
#pragma unroll
        for (int sg = 0; sg < kSegPerWave; ++sg) x[sg] = load(row, at[sg]);
    });
#pragma unroll
    for (int sg = 0; sg < kSegPerWave; ++sg) mask_group(x[sg], at[sg], v[sg]);
#pragma unroll
    for (int sg = 0; sg < kSegPerWave; ++sg) {
        const int seg = c * kSegPerChunk + wave + sg * kWavesPerBlock;
        if (greedy) {
            ArgMax am{-INFINITY, 0x7fffffff};
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (at[sg] + e >= v[sg] && at[sg] + e < V) am = argmax_merge(am, ArgMax{f4get(x[sg], e), at[sg] + e});
            am = wave_argmax(am);
            if (lane == 0 && seg < NSEG) { publish_store(&rec0[seg], (double)am.v); publish_store(&rec1[seg], (double)am.i); }
        } else {
            float mx = -INFINITY;
#pragma unroll
            for (int e = 0; e < 4; ++e) mx = fmaxf(mx, f4get(x[sg], e) * invT);
            mx = wave_max(mx);
            float acc = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float st = f4get(x[sg], e) * invT;
                if (st > -INFINITY) acc += __expf(st - mx);
            }
            const double sum = (double)wave_sum(acc);
            if (lane == 0 && seg < NSEG) { publish_store(&rec0[seg], sum); publish_store(&rec1[seg], (double)mx); }
        }
    }
    publish_barrier();
    if (tid == 0) s_last = arrive(&a.tickets[(size_t)b * a.TS], (uint32_t)a.C5) ? 1 : 0;
    __syncthreads();
    if (!s_last) return;

    const size_t fidx = (size_t)b * (gamma + 1) + k;
    const int SPT = (NSEG + kBlock - 1) / kBlock;
    const int g0 = min(NSEG, tid * SPT), g1 = min(NSEG, g0 + SPT);
    const int leaf_tok = a.sib_tokens[so];
    if (greedy) {
        ArgMax am{-INFINITY, 0x7fffffff};
        for (int g = g0; g < g1; ++g) am = argmax_merge(am, ArgMax{(float)published_load(&rec0[g]), (int)published_load(&rec1[g])});
        am = wave_argmax(am);
        if (lane == 0) s_am[wave] = am;
        __syncthreads();
        if (tid == 0) {
            ArgMax t = s_am[0];
            for (int w = 1; w < kWavesPerBlock; ++w) t = argmax_merge(t, s_am[w]);
            a.out_tokens[fidx] = leaf_tok;
            a.out_tokens[fidx + 1] = (t.i >= 0 && t.i < V) ? t.i : 0;
            a.flags[fidx + 1] = 0;
            a.leaf[b] = sidx;
            a.n_out[b] = k + 2;
            ts[kTsStatus] = (double)kTreeDone;
        }
        return;
    }
    if (tid == 0) a.flags[fidx] = (uint8_t)w.flag;
    float ml = -INFINITY;
    for (int g = g0; g < g1; ++g) ml = fmaxf(ml, (float)published_load(&rec1[g]));
    const float M = block_max(ml, s_redf);
    double run = 0.0;
    for (int g = g0; g < g1; ++g) {
        const double sg = published_load(&rec0[g]);
        if (sg > 0.0) run += sg * exp(published_load(&rec1[g]) - (double)M);
    }
    // rescaled masses go back to slot 0 so that the owner can walk its own run (only this workgroup is left)
    double Z;
    const double excl = block_exclusive_scan(run, s_redd, &Z);
    const float u = a.u_res ? a.u_res[b] : tabed_uniform(a.seed, a.round, (uint32_t)b, (uint32_t)gamma, 0);
    const double target = (double)u * Z;
    uint32_t flag = 0;
    const int owner = block_find_owner(excl, run, target, s_first, s_lastw);
    if (owner < 0) {
        if (tid == 0) {
            a.out_tokens[fidx] = leaf_tok; a.out_tokens[fidx + 1] = 0;
            a.flags[fidx + 1] = (uint8_t)(TABED_FLAG_SAMPLE_MARGIN | TABED_FLAG_DEGENERATE);
            a.leaf[b] = sidx; a.n_out[b] = k + 2; ts[kTsStatus] = (double)kTreeDone;
        }
        return;
    }
    if (tid == owner) {
        double P = excl, Plast = excl;
        int gstar = -1, glast = g0;
        for (int g = g0; g < g1; ++g) {
            const double sg = published_load(&rec0[g]);
            const double mg = (sg > 0.0) ? sg * exp(published_load(&rec1[g]) - (double)M) : 0.0;
            if (mg > 0.0) { glast = g; Plast = P; }
            if (P + mg > target) { gstar = g; break; }
            P += mg;
        }
        if (gstar < 0) { gstar = glast; P = Plast; }
        s_seg = gstar;
        s_prefix = P;
    }
    __syncthreads();
    if (tid >= kWave) return;
    const int v1 = s_seg * kSegV + lane * 4, at1 = group_at(v1, V);
    float4 xx;
    with_row_loads(V, [&](auto load) { xx = load(row, at1); });
    mask_group(xx, at1, v1);
    float f[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float st = f4get(xx, e) * invT;
        f[e] = (st > -INFINITY) ? __expf(st - M) : 0.f;
    }
    const int tok = tree_pick_token(f, at1, V, s_prefix, target, Z, &flag);
    if (lane == 0) {
        a.out_tokens[fidx] = leaf_tok;
        a.out_tokens[fidx + 1] = tok;
        a.flags[fidx + 1] = (uint8_t)flag;
        a.leaf[b] = sidx;
        a.n_out[b] = k + 2;
        ts[kTsStatus] = (double)kTreeDone;
    }
}

// The next pass of every sequence.  first: of the walk, which starts here.
template <int N>
__global__ __launch_bounds__(kBlock) void k_tree_pass(TreeArgs a, int first) {
    const int c = blockIdx.x, b = blockIdx.y;
    double* ts = a.tstate + (size_t)b * kTsSlots;
    TreeWalk w;
    if (first) {
        w = tree_begin(a, b);
        if (w.status == kTreeDone && c == 0 && threadIdx.x == 0) {
            a.leaf[b] = 0;
            a.n_out[b] = w.k + 1;
            ts[kTsStatus] = (double)kTreeDone;              // (nobody reads it in this launch)
        }
    } else {
        w.status = __builtin_amdgcn_readfirstlane((int)ts[kTsStatus]);
        if (w.status == kTreeDone) return;
        w.index = __builtin_amdgcn_readfirstlane((int)ts[kTsIndex]);
        w.k = __builtin_amdgcn_readfirstlane((int)ts[kTsK]);
        w.flag = a.flags[(size_t)b * (a.gamma + 1) + w.k];
    }
    if (w.status == kTreePending) tree_level<N>(a, c, b, w);
    else if (w.status == kTreeLeaf) tree_bonus(a, c, b, w);
}

hipError_t launch_verify_tree(const tabed_cfg& c, const WsLayout& L, char* ws, uint64_t round, int width,
                              const float* target_logits, const float* leaf_logits, const float* draft_logits,
                              const double* draft_lse, const int32_t* sib_tokens, const float* sib_q,
                              const float* weights, const float* temperature, const float* u_res,
                              const float* u_acc_sib, int32_t* out_tokens, uint8_t* flags, int32_t* leaf,
                              int32_t* n_out, hipStream_t s) {
    ProfScope prof(TABED_K_TREE, s);
    TreeArgs a;
    a.V = c.V; a.n = c.n; a.B = c.B; a.gamma = c.gamma; a.S = width - 1; a.NSEG = L.NSEG; a.C5 = L.C5; a.TS = L.TS;
    a.seed = c.seed; a.round = round;
    a.target = target_logits; a.leaf_logits = leaf_logits; a.dlogits = draft_logits; a.dlse = draft_lse;
    a.sib_tokens = sib_tokens; a.sib_q = sib_q; a.weights = weights; a.temperature = temperature;
    a.u_res = u_res; a.u_acc_sib = u_acc_sib;
    a.tstate = reinterpret_cast<double*>(ws + L.off_tstate);
    a.segP = reinterpret_cast<const double*>(ws + L.off_seg);
    a.tseg = reinterpret_cast<double*>(ws + L.off_tseg);
    a.out_tokens = out_tokens; a.flags = flags; a.leaf = leaf; a.n_out = n_out;
    a.tickets = reinterpret_cast<uint32_t*>(ws + L.off_tickets) + 3 * (size_t)c.B * L.TS;
    const int ncomp = compiled_drafts(c.n);
    for (int pass = 0; pass < std::max(1, width - 1); ++pass) {      // (width 1: no sibling, leaf = 0 and n_out = k + 1)
        const dim3 grid(width == 1 ? 1 : L.C5, c.B);
#define TABED_PASS(N_) launch(pass == 0 ? &prof : nullptr, k_tree_pass<N_>, grid, dim3(kBlock), 0, s, a, pass == 0 ? 1 : 0)
        TABED_FOR_DRAFTS(ncomp, TABED_PASS)
#undef TABED_PASS
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace tabed
