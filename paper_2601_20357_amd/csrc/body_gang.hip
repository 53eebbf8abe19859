// The draft-model body's decode step as ONE launch, for the row counts where its launches, not its bytes, were the time: up to
// 16 rows (gang_applies).  256 workgroups of 512 threads, one per compute unit,
// walk the layers together; a layer is five phases (q/k/v, attention, output projection, gate / up, down) whose items are
// dealt to the workgroups.
//
// What bounds it.  With few rows a projection moves 1 to 9 MB, 0.2 to 1.4 us for the chip, and as a launch of its own takes 5
// to 7: 1.5 us of dispatch, 2.6 us until the first dependent load is back, and W behind it.  Here a workgroup has the weights
// (or keys and values) of its next item in registers before what the item depends on exists, and what crosses
// workgroups announces itself: a result is stored past the caches over words that hold a pattern no result has, and whoever
// needs it reads it, past the caches too, until none of the pattern is left.  That is one trip of 0.5 us between two
// workgroups (measured as a ping-pong), where stores that are waited for, arrival counters, a poll and then the first load
// took 2.2 us with 256 workgroups, and a kernel boundary more.  With 48 to 192 writers and as many readers a hand-over is 1.3 to
// 1.9 us from the store to the last reader, and a layer has five: that bounds it now.  One step of 12 layers, d = 768, d_ff = 3072,
// 4 rows of 600 to 1900 positions: 228 us, 336 as 62 launches; one layer 19 us, 28.
//
// Why nothing can wait for ever.  A workgroup only waits for workgroups that are running: at the start each registers, the
// registration is closed when all have come or after a bounded time, whoever comes later leaves at once, and the items are
// dealt to those that are in (P of them).  So neither another kernel that holds compute units nor a second step on another
// stream can stop it; with fewer workgroups it is slower.  Beside a stream of matrix products, step / product in us, one launch and
// launches: 12 layers as above and products of 25 us that fill part of the chip 295 / 43 and 367 / 30, of 790 us that fill it
// 785 / 956 and 1223 / 825; two layers 71 / 33 and 66 / 29, 242 / 845 and 253 / 842.  Results do not depend on P: items are fixed, and only who
// computes them varies.  Should a wait go unanswered all the same, it ends after some time, and what it waited for is taken as it
// is, a NaN, so that those who wait for what follows from it are answered.  The step says so: H has the NaN, the positions stay, and
// the next launch fills the buffers anew.
//
// Why a result is whole.  Every buffer has its own place in every layer and is written once a launch.  There are two sets of
// buffers, used in turn: a launch fills the other set with the pattern for the next one (the end of a launch orders that).
// The control block says which set is next and for which sizes they were filled; where the workspace was used for
// something else in between, all fill both sets and wait for one another first.  A pattern is recognised per stored piece
// of 4 or 8 bytes.  A control block that was never prepared, or was written over, is known by a mark that only the preparation
// writes: nothing in it can be relied on, so the first workgroup does all of the step by itself, which takes milliseconds and
// is right.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "body_utils.h"
#include "device_utils.h"
#include "internal.h"

namespace tabed {

constexpr int kGangGroups = 256, kGangThreads = 512, kGangWaves = 8;
constexpr int kGangChunk = 32;                       // keys: granule in which attention is cut into pieces
constexpr uint32_t kClosedHi = 0x80000000u;          // upper half of a registration word
// control block, in 128-byte lines: registration (8), what it was when closed (8), exit count, arrivals at the one common wait
// (8), and, kept from launch to launch, the state of the buffers (their key and which of the two sets comes next) and the mark
// of a block that has been prepared
constexpr int kLineReg = 0, kLineFinal = 8, kLineExit = 16, kLineArrive = 17, kLineState = 25, kLines = 26;
static_assert(kLines * 128 <= (int)kGangControlBytes, "control block");
constexpr uint64_t kPrepared = 0x9e3779b97f4a7c15ull;

struct GangArgs {
    int rows, layers, d, heads, d_ff, V, max_ctx;
    float eps;
    double log2_theta;
    const int32_t* token_src;
    int token_stride, rows_per_token;
    int32_t* ctx_len;
    uint16_t* kcache;
    uint16_t* vcache;
    uint16_t* H;
    uint32_t* ctl;
    char* buf;                                       // two sets; layer l of a set at l * layer_bytes
    uint32_t layer_bytes, set_bytes;
    int late_from, absent;                           // for tests: workgroups from late_from on come late, and one that does nothing
    uint64_t key;                                    // the sizes that the buffers' place and layout follow from
    uint32_t off_q, off_kn, off_vn, off_po, off_att, off_xa, off_act, off_xm;
    tabed_body_weights w;
};

// What a word is filled with: a NaN that no instruction makes; one that came in with the inputs is stored as another.
constexpr uint32_t kUnset = 0xffffffffu;
__device__ __forceinline__ uint32_t announced(uint32_t v) { return v == kUnset ? 0x7fffffffu : v; }
__device__ __forceinline__ void announce64(void* p, uint32_t lo, uint32_t hi) {
    __hip_atomic_store(reinterpret_cast<uint64_t*>(p), (uint64_t)announced(lo) | ((uint64_t)announced(hi) << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void announce_f4(void* p, float a, float b, float c, float d) {
    announce64(p, __builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b));
    announce64(static_cast<char*>(p) + 8, __builtin_bit_cast(uint32_t, c), __builtin_bit_cast(uint32_t, d));
}
__device__ __forceinline__ bool unset(const u32x4b& v) { return v[0] == kUnset || v[1] == kUnset || v[2] == kUnset || v[3] == kUnset; }

// v combined with the v of the lane 16, or 32, away.  (The results are copied out first: a bit cast of an element of the
// returned vector reads element 0.)
template <typename F>
__device__ __forceinline__ float with_lane16(float v, F f) {
    const uint32_t x = __builtin_bit_cast(uint32_t, v);
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    const uint32_t r0 = r[0], r1 = r[1];
    return f(__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1));
}
template <typename F>
__device__ __forceinline__ float with_lane32(float v, F f) {
    const uint32_t x = __builtin_bit_cast(uint32_t, v);
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const uint32_t r0 = r[0], r1 = r[1];
    return f(__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1));
}
__device__ __forceinline__ float add_lanes16_32(float v) {
    auto add = [](float p, float q) { return p + q; };
    return with_lane32(with_lane16(v, add), add);
}
__device__ __forceinline__ float max_lanes16_32(float v) {
    auto larger = [](float p, float q) { return fmaxf(p, q); };
    return with_lane32(with_lane16(v, larger), larger);
}
constexpr int kDppRor8 = 0x128;                      // row_ror:8 = lane ^ 8 within 16

__device__ __forceinline__ void keep_order() { asm volatile("" ::: "memory"); }

// Every wait is answered; a bound all the same, of some tenths of a second.  (What is then taken as it is counts as announced
// where it is used, so that only those who wait for a workgroup that is lost itself come to it, once a phase.)
constexpr int kMaxSpins = 1 << 18;
constexpr uint32_t kGaveUp = 0x10000u;               // in the exit count, for each workgroup in which one has

// LPK: lanes per key (head_dim / 8).  UD, UF: units of 32 of the contraction over d and over d_ff that a wave takes, at most.
template <int LPK, int UD, int UF>
__global__ __launch_bounds__(kGangThreads, 2) void k_body_gang(GangArgs a) {
    constexpr int hd = LPK * 8, half_hd = hd / 2, TPH = hd / 32;            // TPH: pairs of 16-column tiles per head
    constexpr int kPatchRow = 80, kPatch = 16 * kPatchRow;
    constexpr int kRec = hd * 4 + 16;                                       // a piece of attention: sums, maximum, sum of p
    extern __shared__ __attribute__((aligned(16))) unsigned char s_dyn[];   // (its size keeps a second workgroup off the compute unit)
    __shared__ int s_pos[16], s_tok[16], s_np[16], s_pre[17], s_id, s_P, s_set, s_known, s_solo, s_gave_up;
    __shared__ float s_ml[2][kGangWaves][2];
    __shared__ __attribute__((aligned(16))) float s_ss[16][12], s_o[2][kGangWaves][hd];
    __shared__ __attribute__((aligned(16))) float s_part[kGangWaves][2][64][4];
    __shared__ __attribute__((aligned(16))) unsigned char s_patch[kGangWaves][kPatch], s_junk[kGangWaves][256];
    double2* const s_trig = reinterpret_cast<double2*>(s_dyn);              // [rows][hd/2]

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int lane = tid & 63, r16 = lane & 15, c = lane >> 4;
    int rows = a.rows, d = a.d, heads = a.heads, dff = a.d_ff;
    int TD = d >> 4, units_d = d >> 5, TF = (dff + 15) >> 4, rowc = min(r16, rows - 1);
    // what follows from these is computed anew in every phase: kept in registers across the phases it spilled
    auto new_phase = [&]() {
        asm volatile("" : "+v"(lane), "+s"(rows), "+s"(d), "+s"(heads), "+s"(dff));
        r16 = lane & 15; c = lane >> 4;
        TD = d >> 4; units_d = d >> 5; TF = (dff + 15) >> 4;
        rowc = min(r16, rows - 1);                                          // rows that are not there: one that is
    };
    uint32_t* const ctl = a.ctl;
    if ((int)blockIdx.x >= a.late_from) {                                   // (tests: when the registration is closed, 3 ms)
        const uint64_t began = __builtin_amdgcn_s_memrealtime();
        while (__builtin_amdgcn_s_memrealtime() - began < 300000) __builtin_amdgcn_s_sleep(8);
    }

    // ---- registration: a bit of the workgroup's own in one of eight words.  Normally all come at once and their numbers are
    //      their ids.  Whoever has waited too long closes the words, which settles who is in: the first to close a word
    //      writes down what it held, and the ids are the ranks in that.
    uint64_t before = 0;
    if (tid == 0) s_gave_up = 0;
    if (tid == 0)
        before = __hip_atomic_fetch_or(reinterpret_cast<uint64_t*>(ctl + (kLineReg + (blockIdx.x & 7)) * 32), 1ull << (blockIdx.x >> 3),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // ---- positions and tokens.  (The positions move on when all workgroups have left: one that read them later would cut the
    //      attention into other pieces than the rest, and could wait for pieces that nobody computes.)
    if (wave == 1) {
        const int r = min(lane, rows - 1);
        const int pos = min(max(a.ctx_len[r], 0), a.max_ctx - 1);
        const int tok = a.token_src[(size_t)(r / a.rows_per_token) * a.token_stride];
        // Attention is cut into pieces: a row's and head's keys into np parts of about equal length, none longer than z chunks; z
        // is the smallest that gives no more pieces than workgroups (rows * heads <= 256), and at most 8 of a row and head, or 16
        // where they have 256 keys and more: one wave merges them eight at a time (without that limit one layer of one head of
        // 64, one row of 7000 positions 41.5 us, 23.7 with 16; of 600 to 1900 25.5, 21.6 with 8; as launches 22.6 and 19.6).
        const int nch = (lane < rows) ? pos / kGangChunk + 1 : 0;
        auto row_sum = [](int x) {
            x += dpp_i32<kDppXor1>(x); x += dpp_i32<kDppXor2>(x); x += dpp_i32<kDppHalfMirror>(x); x += dpp_i32<kDppMirror>(x);
            return __builtin_amdgcn_readfirstlane(x);                       // rows are in the first 16 lanes
        };
        int z0 = 1, z1 = 8192 / kGangChunk;
        while (z0 < z1) {
            const int z = (z0 + z1) >> 1;
            const int n = (nch + z - 1) / z;
            if (row_sum(n) * heads <= kGangGroups && __all(n <= (z >= 8 ? 16 : 8))) z1 = z;
            else z0 = z + 1;
        }
        const int np = (nch + z0 - 1) / z0;
        int inc = np;                                                       // prefix over the rows
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const int t = __shfl_up(inc, o);
            inc += (lane >= o) ? t : 0;
        }
        if (lane < 16) {
            s_pos[lane] = pos;
            s_tok[lane] = min(max(tok, 0), a.V - 1);
            s_np[lane] = np;
            s_pre[lane + 1] = inc;
        }
        if (lane == 0) s_pre[0] = 0;
    }
    if (tid == 2 * kWave) {                                                 // the last workgroup of a launch changes it, when all are through
        const uint64_t* state = reinterpret_cast<const uint64_t*>(ctl + kLineState * 32);
        s_known = __hip_atomic_load(state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.key;
        s_set = (int)(__hip_atomic_load(state + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1);
        s_solo = __hip_atomic_load(state + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != kPrepared;      // (no launch changes that)
    }
    __syncthreads();
    // (in the shadow of the others' arrival) rotation angles of all rows, in fp64: a position times a tiny frequency loses digits in fp32
    for (int i = tid; i < rows * half_hd; i += kGangThreads) {
        double sn, cs;
        sincos((double)s_pos[i / half_hd] * exp2(-2.0 * (double)(i % half_hd) / (double)hd * a.log2_theta), &sn, &cs);
        s_trig[i] = make_double2(cs, sn);
    }
    const bool solo = __builtin_amdgcn_readfirstlane(s_solo) != 0;
    if (solo && tid == 0) { s_id = 0; s_P = (blockIdx.x == 0) ? 1 : 0; }
    if (wave == 0 && !solo) {
        constexpr int per = kGangGroups / 8;                                // bits of a word
        constexpr uint64_t full = (1ull << per) - 1;
        uint64_t* const words = reinterpret_cast<uint64_t*>(ctl + (kLineReg + (lane & 7)) * 32);
        uint64_t* const finals = reinterpret_cast<uint64_t*>(ctl + (kLineFinal + (lane & 7)) * 32);
        const bool late = ((uint32_t)__builtin_amdgcn_readfirstlane((int)(before >> 32)) & kClosedHi) != 0;
        int P = 0, id = 0;
        const uint64_t began = __builtin_amdgcn_s_memrealtime();            // 100 MHz
        bool closed = false;
        while (!late) {
            const uint64_t w = __hip_atomic_load(words, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (__all(w == full)) { P = kGangGroups; id = (int)blockIdx.x; break; }
            if (__any((w >> 32) != 0)) closed = true;                       // somebody closes: so do I, until all words are
            const uint64_t waited = __builtin_amdgcn_s_memrealtime() - began;
            int in = (lane < 8) ? __popcll(w & full) : 0;
            in += dpp_i32<kDppXor1>(in); in += dpp_i32<kDppXor2>(in); in += dpp_i32<kDppHalfMirror>(in);
            in = __builtin_amdgcn_readfirstlane(in);
            if (closed || (waited > 2000 && in >= kGangGroups / 4) || waited > 100000) {      // 20 us with a quarter of them, 1 ms with any
                if (lane < 8) {
                    const uint64_t old = __hip_atomic_fetch_or(words, (uint64_t)kClosedHi << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((old >> 32) == 0) __hip_atomic_store(finals, old | ((uint64_t)kClosedHi << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                uint64_t f = 0;
                bool all = false;
                for (int spin = 0; spin < kMaxSpins && !all; ++spin) {      // (the first to close a word writes it down right away)
                    f = __hip_atomic_load(finals, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    all = __all((f >> 32) != 0);
                }
                if (!all) {                                                 // takes no part
                    if (lane == 0) s_gave_up = 1;
                    break;
                }
                const uint32_t bit = blockIdx.x >> 3;
                for (int q = 0; q < 8; ++q) {                               // rank among those who are in, in the order of their numbers
                    const uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)f, q);
                    id += __popc(bits & ((1u << bit) - 1u)) + ((q < (int)(blockIdx.x & 7)) ? (int)((bits >> bit) & 1u) : 0);
                    P += __popc(bits);
                }
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        if (id == a.absent) P = 0;
        if (lane == 0) { s_id = id; s_P = P; }
    }
    __syncthreads();
    const int P = s_P, id = s_id;
    if (P > 0) {
        const int set = __builtin_amdgcn_readfirstlane(s_set);
        const bool known = s_known != 0 && !solo;
        for (int which = known ? 1 : 0; which < 2; ++which) {
            char* const to = a.buf + (size_t)(set ^ which) * a.set_bytes;
            for (uint32_t o = ((uint32_t)id * kGangThreads + tid) * 16u; o < a.set_bytes; o += (uint32_t)P * kGangThreads * 16u) {
                if (known) {
                    *reinterpret_cast<u32x4b*>(to + o) = u32x4b{kUnset, kUnset, kUnset, kUnset};
                } else {
                    __hip_atomic_store(reinterpret_cast<uint64_t*>(to + o), ~0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(reinterpret_cast<uint64_t*>(to + o) + 1, ~0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        if (!known) {
            publish_barrier();
            if (wave == 0 && !solo) {
                if (lane == 0) __hip_atomic_fetch_add(ctl + (kLineArrive + (id & 7)) * 32, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const int want = (P - (lane & 7) + 7) >> 3;
                bool all = false;
                for (int spin = 0; spin < kMaxSpins && !all; ++spin) {
                    const int v = (int)__hip_atomic_load(ctl + (kLineArrive + (lane & 7)) * 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    all = __all(v >= want);
                    if (!all) __builtin_amdgcn_s_sleep(1);
                }
                if (!all) {                                                 // takes no part: what stands in the buffers may be anything
                    if (lane == 0) { s_gave_up = 1; s_P = 0; }
                }
            }
            __syncthreads();
            if (s_P == 0 && id == 0)
                for (uint32_t i = tid; i < (uint32_t)(rows * d) / 2; i += kGangThreads) reinterpret_cast<uint32_t*>(a.H)[i] = 0x7fff7fffu;
        }
    }
    if (s_P > 0) {
        const int set = __builtin_amdgcn_readfirstlane(s_set);
        if (id == 0 && tid == 0) __hip_atomic_store(ctl + kLineState * 32 + 6, (uint32_t)P, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);     // (for tests)
        char* const buf = a.buf + (size_t)set * a.set_bytes;
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(buf, 0, (int)a.set_bytes, 0x00020000);
        auto coherent16 = [&](uint32_t off) { return __builtin_bit_cast(u32x4b, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 16)); };   // sc1
        auto as_f4 = [](const u32x4b& v) { return __builtin_bit_cast(f32x4b, v); };
        int waited = 0;                                                     // kMaxSpins is in it if a wait of this wave went unanswered
        // load() requests, and says whether anything is missing still
        auto until_set = [&](auto load) {
            int spin = 0;
            bool missing;
#pragma nounroll
            do {
                keep_order();
                missing = __any(load());
            } while (missing && ++spin < kMaxSpins);
            waited = __builtin_amdgcn_readfirstlane(waited | spin);         // (a branch here, or an LDS store, cost 3 % of a step)
        };
        // Where many wait for the same data, each wave watches one piece of it, of row 0, before it asks for all of its share: 192
        // workgroups that asked for everything time and again kept the stores of what they waited for from getting through (a
        // step of 12 layers 6 us longer).  Measured and not kept: a word per item, behind its result, that one wave of a
        // workgroup watches, and the results then through the caches (58 us longer).
        auto glance = [&](uint32_t off) { until_set([&]() { return r16 == 0 && unset(coherent16(off)); }); };
        const int pieces = s_pre[16] * heads;                               // of attention
        const int off3 = P * 3 / 4;                                         // output and down projections start where gate / up leaves room
        auto first_of = [&](int off) { const int i = id - off; return i < 0 ? i + P : i; };
        unsigned char* const patch = s_patch[wave];
        // W, 16 rows of 32 k: four lanes a row, requested here, turned through the wave's patch into operand layout later
        auto request_w = [&](u32x4b& raw, const uint16_t* wrow0, int last_row, int K, int unit) {
            const uint32_t row = (uint32_t)min(lane >> 2, last_row);
            const uint32_t k = (uint32_t)min(unit * 32 + (lane & 3) * 8, K - 8);
            raw = *reinterpret_cast<const u32x4b*>(reinterpret_cast<const char*>(wrow0) + (row * (uint32_t)K + k) * 2u);
        };
        auto turn_w = [&](const u32x4b& raw) {                              // LDS operations of one wave execute in order: no barrier
            *reinterpret_cast<u32x4b*>(patch + (lane >> 2) * kPatchRow + (lane & 3) * 16) = raw;
            return *reinterpret_cast<const bf16x8*>(patch + r16 * kPatchRow + c * 16);
        };
        // brings lines of W into the L2 long before request_w: one word of each goes to a corner of LDS that nobody reads
        auto touch = [&](const uint16_t* w, int rows_of_w, int K) {
            const uint32_t bytes = (uint32_t)rows_of_w * (uint32_t)K * 2u;
            for (uint32_t o = 0; o < bytes; o += kGangThreads * 128u) {
                const uint32_t at = min(o + (uint32_t)(wave * 64 + lane) * 128u, bytes - 4u);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(reinterpret_cast<const char*>(w) + at),
                                                 (__attribute__((address_space(3))) void*)s_junk[wave], 4, 0, 0);
            }
        };
        auto touch_layer = [&](int l) {
            new_phase();
            for (int it = first_of(0); it < 3 * units_d; it += P) {
                const int part = it / units_d, t = it % units_d;
                const uint16_t* w = static_cast<const uint16_t*>(a.w.wqkv[l]) + (size_t)(part * d + t / TPH * hd + (t % TPH) * 16) * d;
                touch(w, 16, d);
                touch(w + (size_t)half_hd * d, 16, d);
            }
            for (int it = first_of(off3); it < TD; it += P) {
                touch(static_cast<const uint16_t*>(a.w.wo[l]) + (size_t)it * 16 * d, 16, d);
                touch(static_cast<const uint16_t*>(a.w.wdown[l]) + (size_t)it * 16 * dff, 16, dff);
            }
            for (int it = first_of(0); it < TF; it += P) {
                const uint16_t* w = static_cast<const uint16_t*>(a.w.wgu[l]) + (size_t)it * 16 * d;
                touch(w, min(16, dff - it * 16), d);
                touch(w + (size_t)dff * d, min(16, dff - it * 16), d);
            }
        };
        // the waves' partial results of tile nb, added in wave order
        auto total = [&](int nb) {
            f32x4b t = *reinterpret_cast<const f32x4b*>(s_part[0][nb][lane]);
#pragma unroll
            for (int w = 1; w < kGangWaves; ++w) t += *reinterpret_cast<const f32x4b*>(s_part[w][nb][lane]);
            return t;
        };
        auto embed4 = [&](int row, int col) {
            const uint2 e = *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(a.w.embed) + (size_t)s_tok[row] * d + col);
            return f32x4b{__builtin_bit_cast(float, e.x << 16), __builtin_bit_cast(float, e.x & 0xffff0000u),
                          __builtin_bit_cast(float, e.y << 16), __builtin_bit_cast(float, e.y & 0xffff0000u)};
        };
        // Activations are kept the way the next matrix product takes them, so that a wave reads contiguous pieces: lane (r16, c)
        // of a wave takes, of row r16, the eight columns from 8 c of a unit of 32.
        //   residual stream, fp32: [unit][half of the eight][c][row][4];  bf16: [unit][c][row][8]
        // Where the four columns from 4 c of tile `tile`, which a finishing lane holds, go (bytes):
        auto x_at = [&](int tile) { return (uint32_t)((((tile >> 1) * 2 + (c & 1)) * 4 + (tile & 1) * 2 + (c >> 1)) * rows + rowc) * 16u; };

        touch_layer(0);
        for (int l = 0; l < a.layers; ++l) {
            const uint32_t lo = (uint32_t)l * a.layer_bytes, x_before = lo + a.off_xm - a.layer_bytes;      // (l > 0)
            char* const lb = buf + lo;
            uint16_t* const kc = a.kcache + (size_t)l * rows * a.max_ctx * d;
            uint16_t* const vc = a.vcache + (size_t)l * rows * a.max_ctx * d;

            // ---- attention's first keys and values: nothing of this step is needed for them
            constexpr int U = 4, GK = kWave / LPK, kStep = kGangWaves * GK * U;
            struct Piece { int v, r, h, t0, t1, fresh; };                   // keys t0 <= t < t1 of the cache; fresh: and the new position's
            auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
            auto piece_at = [&](Piece& s, int v) {                          // uniform
                const int r = __popcll(__ballot(lane < 16 && s_pre[(lane & 15) + 1] * heads <= v));
                const int np = uni(s_np[r]), rem = v - uni(s_pre[r]) * heads, pos = uni(s_pos[r]), nch = pos / kGangChunk + 1;
                const int h = uni((int)((uint32_t)rem / (uint32_t)np)), i = rem - h * np;
                s.v = v; s.r = r; s.h = h;
                s.t0 = uni((int)((uint32_t)(i * nch) / (uint32_t)np)) * kGangChunk;
                s.t1 = min(uni((int)((uint32_t)((i + 1) * nch) / (uint32_t)np)) * kGangChunk, pos);
                s.fresh = (i == np - 1);
            };
            auto request_kv = [&](u32x4b (&k4)[U], u32x4b (&v4)[U], const Piece& s, int t) {
                const size_t base = (size_t)s.r * a.max_ctx * d + s.h * hd;
                const char* const kb = reinterpret_cast<const char*>(kc + base);
                const char* const vb = reinterpret_cast<const char*>(vc + base);
                const int last = max(s.t1 - 1, 0), first = t + wave * GK + lane / LPK;      // past the end: the last one again
                uint32_t o[U];
#pragma unroll
                for (int u = 0; u < U; ++u) o[u] = (uint32_t)(min(first + u * kGangWaves * GK, last) * d + lane % LPK * 8) * 2u;
#pragma unroll
                for (int u = 0; u < U; ++u) k4[u] = *reinterpret_cast<const u32x4b*>(kb + o[u]);
#pragma unroll
                for (int u = 0; u < U; ++u) v4[u] = *reinterpret_cast<const u32x4b*>(vb + o[u]);
            };
            Piece pc{};
            u32x4b kw[U], vw[U];
            new_phase();
            if (id < pieces) {
                piece_at(pc, id);
                request_kv(kw, vw, pc, pc.t0);
            }
            keep_order();

            // RMSNorm + projection onto two 16-column tiles; leaves the waves' partial results in LDS.  wr0 / wr1: W row of the tiles'
            // first column, last: their last row that exists
            auto normed = [&](const uint16_t* wr0, const uint16_t* wr1, int last, const float* g, bool embed_rows, uint32_t xo) {
                u32x4b raw[2][UD];
                f32x4b gr[UD][2];
#pragma unroll
                for (int u = 0; u < UD; ++u) {
                    const int unit = min(wave + u * kGangWaves, units_d - 1);
                    request_w(raw[0][u], wr0, last, d, unit);
                    request_w(raw[1][u], wr1, last, d, unit);
                }
#pragma unroll
                for (int u = 0; u < UD; ++u) {
                    const int k = min(wave + u * kGangWaves, units_d - 1) * 32 + c * 8;
                    gr[u][0] = *reinterpret_cast<const f32x4b*>(g + k);
                    gr[u][1] = *reinterpret_cast<const f32x4b*>(g + k + 4);
                }
                keep_order();
                bf16x8 w[2][UD];
#pragma unroll
                for (int u = 0; u < UD; ++u) {
                    w[0][u] = turn_w(raw[0][u]);
                    w[1][u] = turn_w(raw[1][u]);
                }
                f32x4b xr[UD][2];
#pragma unroll
                for (int u = 0; u < UD; ++u) {
                    xr[u][0] = f32x4b{0.f, 0.f, 0.f, 0.f};
                    xr[u][1] = f32x4b{0.f, 0.f, 0.f, 0.f};
                }
                if (embed_rows) {
#pragma unroll
                    for (int u = 0; u < UD; ++u) {
                        const int k = min(wave + u * kGangWaves, units_d - 1) * 32 + c * 8;
                        xr[u][0] = embed4(rowc, k);
                        xr[u][1] = embed4(rowc, k + 4);
                    }
                } else {
                    uint32_t at[UD];
#pragma unroll
                    for (int u = 0; u < UD; ++u) at[u] = xo + (uint32_t)((min(wave + u * kGangWaves, units_d - 1) * 8 + c) * rows + rowc) * 16u;
                    const uint32_t half = (uint32_t)rows * 64u;
                    glance(at[UD - 1] + half);
                    until_set([&]() {
                        if (r16 >= rows) return false;                      // (what a wave asks for costs 4 lanes a cycle of the compute unit)
                        u32x4b v[UD][2];
#pragma unroll
                        for (int u = 0; u < UD; ++u) { v[u][0] = coherent16(at[u]); v[u][1] = coherent16(at[u] + half); }
                        bool missing = false;
#pragma unroll
                        for (int u = 0; u < UD; ++u) {
                            missing |= unset(v[u][0]) || unset(v[u][1]);
                            xr[u][0] = as_f4(v[u][0]);
                            xr[u][1] = as_f4(v[u][1]);
                        }
                        return missing;
                    });
                }
                float ss = 0.f;
#pragma unroll
                for (int u = 0; u < UD; ++u) {
                    float t = 0.f;
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const f32x4b v = xr[u][q];
                        t += (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
                    }
                    ss += (wave + u * kGangWaves < units_d) ? t : 0.f;
                }
                ss = add_lanes16_32(ss);
                if (c == 0) s_ss[r16][wave] = ss;
                lds_barrier();                                              // (and the item before is through with s_part)
                const f32x4b s0 = *reinterpret_cast<const f32x4b*>(s_ss[r16]), s1 = *reinterpret_cast<const f32x4b*>(s_ss[r16] + 4);
                ss = ((s0[0] + s0[1]) + (s0[2] + s0[3])) + ((s1[0] + s1[1]) + (s1[2] + s1[3]));
                const float inv = 1.f / sqrtf(ss / (float)d + a.eps);
                f32x4b acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int u = 0; u < UD; ++u) {
                    if (wave + u * kGangWaves < units_d) {                  // uniform
                        const f32x4b v0 = xr[u][0], v1 = xr[u][1], g0 = gr[u][0], g1 = gr[u][1];
                        const uint2 x0 = pack_bf16x4(v0[0] * inv * g0[0], v0[1] * inv * g0[1], v0[2] * inv * g0[2], v0[3] * inv * g0[3]);
                        const uint2 x1 = pack_bf16x4(v1[0] * inv * g1[0], v1[1] * inv * g1[1], v1[2] * inv * g1[2], v1[3] * inv * g1[3]);
                        const bf16x8 xv = __builtin_bit_cast(bf16x8, u32x4b{x0.x, x0.y, x1.x, x1.y});
                        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0][u], xv, acc0, 0, 0, 0);
                        acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[1][u], xv, acc1, 0, 0, 0);
                    }
                }
                *reinterpret_cast<f32x4b*>(s_part[wave][0][lane]) = acc0;
                *reinterpret_cast<f32x4b*>(s_part[wave][1][lane]) = acc1;
                lds_barrier();
            };

            // ================================================================ q/k/v, rotation, cache append
            for (int it = first_of(0); it < 3 * units_d; it += P) {
                new_phase();
                const int part = it / units_d, t = it % units_d, head = t / TPH, j0 = (t % TPH) * 16;
                const uint16_t* wr = static_cast<const uint16_t*>(a.w.wqkv[l]) + (size_t)(part * d + head * hd + j0) * d;
                normed(wr, wr + (size_t)half_hd * d, 15, a.w.g_attn[l], l == 0, x_before);
                if (wave == 0) {                                            // a lane finishes row r16, columns 4 c .. of both tiles
                    f32x4b y0 = total(0), y1 = total(1);
                    if (r16 < rows) {
                        if (part < 2) {
                            f32x4b z0, z1;
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const double2 cs = s_trig[r16 * half_hd + j0 + 4 * c + i];
                                z0[i] = (float)((double)y0[i] * cs.x - (double)y1[i] * cs.y);
                                z1[i] = (float)((double)y1[i] * cs.x + (double)y0[i] * cs.y);
                            }
                            y0 = z0;
                            y1 = z1;
                        }
                        const uint32_t slot = (uint32_t)((head * TPH + j0 / 16) * rows + r16) * 32u + 4u * c;   // [head][tile][row][2 x 16]
                        if (part == 0) {
                            char* q = lb + a.off_q + slot * 4u;
                            announce_f4(q, y0[0], y0[1], y0[2], y0[3]);
                            announce_f4(q + 64, y1[0], y1[1], y1[2], y1[3]);
                        } else {
                            const uint2 b0 = pack_bf16x4(y0[0], y0[1], y0[2], y0[3]), b1 = pack_bf16x4(y1[0], y1[1], y1[2], y1[3]);
                            char* n = lb + (part == 1 ? a.off_kn : a.off_vn) + slot * 2u;
                            announce64(n, b0.x, b0.y);
                            announce64(n + 32, b1.x, b1.y);
                            uint16_t* cache = (part == 1 ? kc : vc) + ((size_t)r16 * a.max_ctx + s_pos[r16]) * d + head * hd + j0 + 4 * c;
                            *reinterpret_cast<uint2*>(cache) = b0;
                            *reinterpret_cast<uint2*>(cache + half_hd) = b1;
                        }
                    }
                }
            }

            // ================================================================ attention over the rows' caches
            // The waves take GK consecutive keys of a piece each in turn, U times a step, requested one step ahead; a piece's partial
            // result (sums, maximum, sum of p) goes to its record.  (The new position's key and value come from the projection, not
            // from the cache, whose lines another XCD's L2 may hold as they were.)
            if (id < pieces) {
                new_phase();
                const int g = lane / LPK, cl = lane % LPK;
                f32x4b qr[2];
                u32x4b knew = {0u, 0u, 0u, 0u}, vnew = {0u, 0u, 0u, 0u};
                auto request_new = [&](f32x4b (&q)[2], u32x4b& k1, u32x4b& v1, const Piece& s) {
                    const int dim = cl * 8, hf = dim >= half_hd, dd = dim - hf * half_hd;
                    const uint32_t o = (uint32_t)((s.h * TPH + dd / 16) * rows + s.r) * 32u + (uint32_t)(hf * 16 + dd % 16);
                    const u32x4b q0 = coherent16(lo + a.off_q + o * 4u), q1 = coherent16(lo + a.off_q + o * 4u + 16u);
                    q[0] = as_f4(q0);
                    q[1] = as_f4(q1);
                    bool missing = unset(q0) || unset(q1);
                    if (s.fresh && wave == 0) {                             // (others do not use them)
                        k1 = coherent16(lo + a.off_kn + o * 2u);
                        v1 = coherent16(lo + a.off_vn + o * 2u);
                        missing |= unset(k1) || unset(v1);
                    }
                    return missing;
                };
                int after = id + P, tb = pc.t0, par = 0;                    // after: the piece after this one
                until_set([&]() { return request_new(qr, knew, vnew, pc); });
                const float scale = 1.44269504f / sqrtf((float)hd);         // scores in base 2
                float m = -FLT_MAX, lsum = 0.f, o[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = 0.f;
                auto dot = [&](const u32x4b& k) {
                    float s = 0.f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        s += (qr[e >> 1][(2 * e) & 3] * scale) * __builtin_bit_cast(float, k[e] << 16);
                        s += (qr[e >> 1][(2 * e + 1) & 3] * scale) * __builtin_bit_cast(float, k[e] & 0xffff0000u);
                    }
                    s += dpp_f32<kDppXor1>(s);
                    s += dpp_f32<kDppXor2>(s);
                    s += dpp_f32<kDppHalfMirror>(s);
                    if (LPK > 8) s += dpp_f32<kDppMirror>(s);
                    return s;
                };
                auto rescale = [&](float mn) {
                    const float keep = __builtin_amdgcn_exp2f(m - mn);
                    m = mn;
                    lsum *= keep;
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] *= keep;
                };
                auto weigh = [&](float s, const u32x4b& v4) {
                    const float p = __builtin_amdgcn_exp2f(s - m);
                    lsum += p;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        o[2 * e] += p * __builtin_bit_cast(float, v4[e] << 16);
                        o[2 * e + 1] += p * __builtin_bit_cast(float, v4[e] & 0xffff0000u);
                    }
                };
                for (bool more = true; more;) {
                    // what comes after this step: the piece's next keys, or the next piece
                    const bool ends = tb + kStep >= pc.t1;
                    f32x4b qn[2] = {qr[0], qr[1]};
                    u32x4b knn = knew, vnn = vnew, kn[U], vn[U];
                    Piece pn = pc;
                    int tbn = tb + kStep;
                    if (ends) {
                        more = after < pieces;
                        if (more) {
                            piece_at(pn, after);
                            tbn = pn.t0;
                            until_set([&]() { return request_new(qn, knn, vnn, pn); });
                        }
                    }
                    if (more) request_kv(kn, vn, pn, tbn);
                    const bool any = tb < pc.t1;                            // (a piece may be the new position alone)
                    float sc[U], mn = m;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const float s = dot(kw[u]);
                        sc[u] = (tb + (u * kGangWaves + wave) * GK + g < pc.t1) ? s : -INFINITY;
                        mn = any ? fmaxf(mn, sc[u]) : mn;
                    }
                    const bool with_new = ends && pc.fresh && wave == 0;    // uniform
                    float scn = -INFINITY;
                    if (with_new) {
                        const float s = dot(knew);
                        scn = (g == 0) ? s : -INFINITY;
                        mn = fmaxf(mn, scn);
                    }
                    rescale(mn);
                    if (any) {
#pragma unroll
                        for (int u = 0; u < U; ++u) weigh(sc[u], vw[u]);
                    }
                    if (with_new) weigh(scn, vnew);
                    if (ends) {
                        // lane groups, then waves, in a fixed order
                        float mw = m;
                        if (LPK <= 8) mw = fmaxf(mw, dpp_f32<kDppRor8>(mw));
                        rescale(max_lanes16_32(mw));
                        auto fold = [&](float x) {
                            if (LPK <= 8) x += dpp_f32<kDppRor8>(x);
                            return add_lanes16_32(x);
                        };
                        lsum = fold(lsum);
#pragma unroll
                        for (int e = 0; e < 8; ++e) o[e] = fold(o[e]);
                        if (lane < LPK) {
                            float* const so = s_o[par][wave];
                            *reinterpret_cast<f32x4b*>(so + lane * 8) = f32x4b{o[0], o[1], o[2], o[3]};
                            *reinterpret_cast<f32x4b*>(so + lane * 8 + 4) = f32x4b{o[4], o[5], o[6], o[7]};
                            if (lane == 0) { s_ml[par][wave][0] = m; s_ml[par][wave][1] = lsum; }
                        }
                        lds_barrier();                                      // (one: the next piece uses the other half of s_o, s_ml)
                        after += P;
                        if (wave == 0) {
                            float M = s_ml[par][0][0], Lt = 0.f, sum[hd / kWave];
#pragma unroll
                            for (int w = 1; w < kGangWaves; ++w) M = fmaxf(M, s_ml[par][w][0]);
#pragma unroll
                            for (int e = 0; e < hd / kWave; ++e) sum[e] = 0.f;
#pragma unroll
                            for (int w = 0; w < kGangWaves; ++w) {
                                const float f = __builtin_amdgcn_exp2f(s_ml[par][w][0] - M);
                                Lt += s_ml[par][w][1] * f;
#pragma unroll
                                for (int e = 0; e < hd / kWave; ++e) sum[e] += s_o[par][w][e * kWave + lane] * f;
                            }
                            char* rec = lb + a.off_po + (uint32_t)pc.v * kRec;
#pragma unroll
                            for (int e = 0; e < hd / kWave; ++e)
                                publish_store(reinterpret_cast<int*>(rec) + e * kWave + lane, (int)announced(__builtin_bit_cast(uint32_t, sum[e])));
                            if (lane == 0) announce64(rec + hd * 4, __builtin_bit_cast(uint32_t, M), __builtin_bit_cast(uint32_t, Lt));
                        }
                        par ^= 1;
                        m = -FLT_MAX;
                        lsum = 0.f;
#pragma unroll
                        for (int e = 0; e < 8; ++e) o[e] = 0.f;
                    }
                    if (more) {
#pragma unroll
                        for (int u = 0; u < U; ++u) { kw[u] = kn[u]; vw[u] = vn[u]; }
                        qr[0] = qn[0]; qr[1] = qn[1];
                        knew = knn; vnew = vnn;
                        pc = pn;
                        tb = tbn;
                    }
                }
                // ---- the workgroup of a row's and head's first piece merges the records of all of them, one wave for the rest, which
                //      go on.  (Merged where they are used, by each of the output projection's tiles, the records took 3 us.)
                if (wave == kGangWaves - 1) {
                    for (int v = id; v < pieces; v += P) {
                        Piece pm;
                        piece_at(pm, v);
                        if (pm.t0 != 0) continue;
                        const int np = uni(s_np[pm.r]);
                        constexpr int E = hd / kWave, NP = 8;               // records requested together
                        float M = -FLT_MAX, Lt = 0.f, t[E];
#pragma unroll
                        for (int e = 0; e < E; ++e) t[e] = 0.f;
                        for (int i0 = 0; i0 < np; i0 += NP) {
                            uint32_t x[NP][E];
                            float2 ml[NP];
                            until_set([&]() {
                                bool missing = false;
#pragma unroll
                                for (int i = 0; i < NP; ++i) {
                                    const uint32_t rec = lo + a.off_po + (uint32_t)(v + min(i0 + i, np - 1)) * kRec;
#pragma unroll
                                    for (int e = 0; e < E; ++e)
                                        x[i][e] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(rec + (uint32_t)(e * kWave + lane) * 4u), 0, 16);
                                    const auto m2 = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(rec + hd * 4), 0, 16);
                                    const uint32_t m0 = m2[0], m1 = m2[1];
                                    missing |= m0 == kUnset || m1 == kUnset;
                                    ml[i] = make_float2(__builtin_bit_cast(float, m0), __builtin_bit_cast(float, m1));
                                }
#pragma unroll
                                for (int i = 0; i < NP; ++i)
#pragma unroll
                                    for (int e = 0; e < E; ++e) missing |= x[i][e] == kUnset;
                                return missing;
                            });
                            float mn = M;
#pragma unroll
                            for (int i = 0; i < NP; ++i) mn = fmaxf(mn, ml[i].x);           // (a record taken twice does not change it)
                            const float keep = __builtin_amdgcn_exp2f(M - mn);
                            M = mn;
                            Lt *= keep;
#pragma unroll
                            for (int e = 0; e < E; ++e) t[e] *= keep;
#pragma unroll
                            for (int i = 0; i < NP; ++i) {
                                const float wgt = (i0 + i < np) ? __builtin_amdgcn_exp2f(ml[i].x - mn) : 0.f;
                                Lt += ml[i].y * wgt;
#pragma unroll
                                for (int e = 0; e < E; ++e) t[e] += __builtin_bit_cast(float, x[i][e]) * wgt;
                            }
                        }
                        const float inv = 1.f / Lt;
#pragma unroll
                        for (int e = 0; e < E; ++e) {
                            const float y = t[e] * inv, z = dpp_f32<kDppXor1>(y);
                            const int k = pm.h * hd + e * kWave + lane;
                            if ((lane & 1) == 0)                            // bf16 activations: [unit][c][row][8]
                                publish_store(reinterpret_cast<int*>(lb + a.off_att + (uint32_t)((k >> 3) * rows + pm.r) * 16u + (uint32_t)(k & 7) * 2u),
                                              (int)announced(pack_bf16x4(y, z, 0.f, 0.f).x));
                        }
                    }
                }
                lds_barrier();                                              // s_o may be written again
            }

            // A projection of bf16 activations at `xo` onto one 16-column tile, added to the residual stream: x_old at `from` (the
            // embedding in the first layer), the sum to `to`
            auto added = [&](auto units_a_wave, const uint16_t* wr, int K, int tile, uint32_t xo, bool embed_rows, uint32_t from, uint32_t to) {
                constexpr int UW = units_a_wave.value;
                const int units = (K + 31) >> 5;
                u32x4b raw[UW];
#pragma unroll
                for (int u = 0; u < UW; ++u) request_w(raw[u], wr, 15, K, min(wave + u * kGangWaves, units - 1));
                keep_order();
                bf16x8 w[UW];
#pragma unroll
                for (int u = 0; u < UW; ++u) w[u] = turn_w(raw[u]);
                f32x4b xold = {0.f, 0.f, 0.f, 0.f};
                if (wave == 0) {
                    if (embed_rows) xold = embed4(rowc, tile * 16 + 4 * c);
                    else until_set([&]() {
                        const u32x4b v = coherent16(from + x_at(tile));
                        xold = as_f4(v);
                        return unset(v);
                    });
                }
                u32x4b xv[UW];
#pragma unroll
                for (int u = 0; u < UW; ++u) xv[u] = u32x4b{0u, 0u, 0u, 0u};
                // (the last whole unit of 32, or, with fewer columns than that, pieces that exist)
                const int watched = min(wave + (UW - 1) * kGangWaves, max(K / 32 - 1, 0)) * 4 + c;
                glance(xo + (uint32_t)(min(watched, K / 8 - 1) * rows) * 16u);
                until_set([&]() {
                    if (r16 >= rows) return false;
                    bool missing = false;
                    const uint32_t at = xo + (uint32_t)(c * rows + r16) * 16u;
#pragma unroll
                    for (int u = 0; u < UW; ++u) xv[u] = coherent16(at + (uint32_t)(min(wave + u * kGangWaves, units - 1) * rows) * 64u);
#pragma unroll
                    for (int u = 0; u < UW; ++u)                            // (columns past K may never be written)
                        missing |= unset(xv[u]) && min(wave + u * kGangWaves, units - 1) * 32 + c * 8 < K;
                    return missing;
                });
                f32x4b acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int u = 0; u < UW; ++u) {
                    const int unit = wave + u * kGangWaves;
                    if (unit < units) {
                        const bool out = unit * 32 + c * 8 >= K;            // K is a multiple of 8: a piece is in or out
                        const u32x4b zero = {0u, 0u, 0u, 0u};
                        const bf16x8 xo8 = __builtin_bit_cast(bf16x8, out ? zero : xv[u]);
                        const bf16x8 wo8 = __builtin_bit_cast(bf16x8, out ? zero : __builtin_bit_cast(u32x4b, w[u]));
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wo8, xo8, acc, 0, 0, 0);
                    }
                }
                lds_barrier();                                              // the item before is through with s_part
                *reinterpret_cast<f32x4b*>(s_part[wave][0][lane]) = acc;
                lds_barrier();
                if (wave == 0) {
                    const f32x4b y = xold + total(0);
                    if (r16 < rows) announce_f4(buf + to + x_at(tile), y[0], y[1], y[2], y[3]);
                }
            };

            // ================================================================ output projection, residual
            for (int tile = first_of(off3); tile < TD; tile += P) {
                new_phase();
                added(std::integral_constant<int, UD>{}, static_cast<const uint16_t*>(a.w.wo[l]) + (size_t)tile * 16 * d, d, tile, lo + a.off_att, l == 0,
                      x_before, lo + a.off_xa);
            }

            // ================================================================ gate / up, SwiGLU
            for (int it = first_of(0); it < TF; it += P) {
                new_phase();
                const uint16_t* wg = static_cast<const uint16_t*>(a.w.wgu[l]) + (size_t)it * 16 * d;
                normed(wg, wg + (size_t)dff * d, min(15, dff - 1 - it * 16), a.w.g_mlp[l], false, lo + a.off_xa);
                if (wave == 0) {
                    const f32x4b gt = total(0), up = total(1);
                    float y[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) y[i] = gt[i] / (1.f + __expf(-gt[i])) * up[i];
                    const uint2 b = pack_bf16x4(y[0], y[1], y[2], y[3]);
                    if (r16 < rows)
                        announce64(lb + a.off_act + (uint32_t)(((it >> 1) * 4 + (it & 1) * 2 + (c >> 1)) * rows + r16) * 16u + (c & 1) * 8u, b.x, b.y);
                }
            }

            // ================================================================ down, residual
            for (int tile = first_of(off3); tile < TD; tile += P) {
                new_phase();
                added(std::integral_constant<int, UF>{}, static_cast<const uint16_t*>(a.w.wdown[l]) + (size_t)tile * 16 * dff, dff, tile, lo + a.off_act,
                      false, lo + a.off_xa, lo + a.off_xm);
            }
            if (l + 1 < a.layers) touch_layer(l + 1);                       // in the shadow of the phases that end the layer
        }

        // ================================================================ final norm
        new_phase();
        const uint32_t xo = (uint32_t)(a.layers - 1) * a.layer_bytes + a.off_xm;
        if (wave == 0) {
            for (int row = id; row < rows; row += P) {
                f32x4b v[4];
                float ss = 0.f;
                uint32_t at[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int k = min((i * 64 + lane) * 4, d - 4);
                    at[i] = xo + (uint32_t)((((k >> 5) * 2 + ((k >> 2) & 1)) * 4 + ((k >> 3) & 3)) * rows + row) * 16u;
                }
                until_set([&]() {
                    bool missing = false;
                    u32x4b t[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) t[i] = coherent16(at[i]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) { missing |= unset(t[i]); v[i] = as_f4(t[i]); }
                    return missing;
                });
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float t = (v[i][0] * v[i][0] + v[i][1] * v[i][1]) + (v[i][2] * v[i][2] + v[i][3] * v[i][3]);
                    ss += ((i * 64 + lane) * 4 < d) ? t : 0.f;
                }
                const float inv = 1.f / sqrtf(wave_sum(ss) / (float)d + a.eps);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int k = (i * 64 + lane) * 4;
                    if (k < d) {
                        const f32x4b g = *reinterpret_cast<const f32x4b*>(a.w.g_final + k);
                        *reinterpret_cast<uint2*>(a.H + (size_t)row * d + k) =
                            pack_bf16x4(v[i][0] * inv * g[0], v[i][1] * inv * g[1], v[i][2] * inv * g[2], v[i][3] * inv * g[3]);
                    }
                }
            }
        }
        if (waited >= kMaxSpins) s_gave_up = 1;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                    // no word is on its way to LDS any more
    }
    lds_barrier();
    // ---- the last workgroup to leave moves the positions on and re-arms the control block for the next launch
    if (tid == 0) {
        auto move_on = [&]() {
            for (int r = 0; r < a.rows; ++r) __hip_atomic_fetch_add(a.ctx_len + r, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        if (s_solo) {
            if (P > 0 && !s_gave_up) move_on();
            return;
        }
        const uint32_t mine = s_gave_up ? kGaveUp : 0u;
        const uint32_t left = __hip_atomic_fetch_add(ctl + kLineExit * 32, 1u + mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((left & (kGaveUp - 1)) == kGangGroups - 1) {
            const bool whole = left < kGaveUp && mine == 0;
            if (whole) move_on();
            uint64_t* state = reinterpret_cast<uint64_t*>(ctl + kLineState * 32);
            __hip_atomic_store(state, whole ? a.key : 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(state + 1, (uint64_t)(s_set ^ 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int i = 0; i < kLineState; ++i)
                __hip_atomic_store(reinterpret_cast<uint64_t*>(ctl + i * 32), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ---------------------------------------------------------------- host side
// Whether a step is one launch.  One launch / a launch per phase, a step in us, rows of 600 to 1900 positions: 12 layers of d = 768,
// d_ff = 3072 at 4 rows 228 / 336, called from the host; replayed in a graph, two such layers 41 / 49 at 1 row, 48 / 56 at 4, 52 / 63 at 8, 63 / 73 at 16; two of d = 256,
// d_ff = 1024 33.0 / 35.2 at 1 row, 39.0 / 50.2 at 16; one of those 20.7 / 20.2 and 23.6 / 24.2.  Called from the host, which takes about 4 us
// a launch, that one layer is 20.9 / 30 and 23.6 / 30, and it is left as one launch, like all the bodies of one layer that a graph would
// replay faster as launches (up to d = 384, by up to 7 %, 1.4 us).  With so many columns that the tiles of gate / up and of the
// output projections do not fit side by side one launch needs more than four rows: two layers of d = 1024, d_ff = 4096 61 / 55 at 1 row, 62 / 60
// at 4, 69 / 73 at 8, 80 / 90 at 16.  (16 rows are one block of the matrix instruction.  From 17 rows on, with counters
// instead of data that announces itself, which so many rows make too much to watch, one launch was slower: 64 rows
// 580 us a block of five steps, 495 as launches.)
bool gang_applies(const tabed_body_cfg& c, int rows) {
    const int hd = c.d / c.heads;
    const bool side_by_side = (c.d_ff + 15) / 16 + c.d / 16 <= kGangGroups;
    return rows <= 16 && (hd == 64 || hd == 128) && c.d <= 1024 && c.d_ff <= 4096 && (side_by_side || rows > 4);
}

struct GangLayout {
    uint32_t off_q, off_kn, off_vn, off_po, off_att, off_xa, off_act, off_xm, layer;
};
static GangLayout gang_layout(const tabed_body_cfg& c, int rows) {
    auto al256 = [](size_t x) { return (uint32_t)((x + 255) / 256 * 256); };
    const size_t R = (size_t)rows, UF = (size_t)(c.d_ff + 31) / 32, hd = c.d / c.heads;
    GangLayout L;
    L.off_q = 0;
    L.off_kn = al256(L.off_q + R * c.d * 4);
    L.off_vn = al256(L.off_kn + R * c.d * 2);
    L.off_po = al256(L.off_vn + R * c.d * 2);
    L.off_att = al256(L.off_po + kGangGroups * (hd * 4 + 16));
    L.off_xa = al256(L.off_att + R * c.d * 2);
    L.off_act = al256(L.off_xa + R * c.d * 4);
    L.off_xm = al256(L.off_act + R * UF * 32 * 2);
    L.layer = al256(L.off_xm + R * c.d * 4);
    return L;
}
size_t gang_bytes(const tabed_body_cfg& c, int rows) { return 2 * (size_t)gang_layout(c, rows).layer * c.layers; }

uint64_t* gang_key(char* ctl) { return reinterpret_cast<uint64_t*>(ctl + kLineState * 128); }

__global__ void k_gang_init(uint32_t* ctl, int words) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    constexpr int mark = kLineState * 32 + 4;                               // the state's third word
    if (i < words) ctl[i] = (i == mark) ? (uint32_t)kPrepared : (i == mark + 1) ? (uint32_t)(kPrepared >> 32) : 0u;
}
hipError_t launch_gang_init(char* ctl, hipStream_t s) {
    const int words = (int)(kGangControlBytes / 4);
    launch(nullptr, k_gang_init, dim3((words + 255) / 256), dim3(256), 0, s, reinterpret_cast<uint32_t*>(ctl), words);
    return hipGetLastError();
}

template <int LPK, int UD, int UF>
static hipError_t launch_gang_t(const GangArgs& a, hipStream_t s) {
    constexpr size_t lds = 84 * 1024;                // the angles take up to 16 KB; as much as keeps workgroups to one a compute unit
    static std::once_flag once;
    static hipError_t rc = hipSuccess;
    if (raise_lds_limit(&k_body_gang<LPK, UD, UF>, lds, once, rc) != hipSuccess) return rc;
    ProfScope prof(TABED_K_BODY, s);
    launch(&prof, k_body_gang<LPK, UD, UF>, dim3(kGangGroups), dim3(kGangThreads), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_gang(const tabed_body_cfg& c, const tabed_body_weights& w, char* ctl, char* buf, int rows, const int32_t* token_src,
                       int token_stride, int rows_per_token, int32_t* ctx_len, uint16_t* kcache, uint16_t* vcache, uint16_t* H, hipStream_t s,
                       int late_from, int absent) {
    const GangLayout L = gang_layout(c, rows);
    GangArgs a{};
    a.rows = rows; a.layers = c.layers; a.d = c.d; a.heads = c.heads; a.d_ff = c.d_ff; a.V = c.V; a.max_ctx = c.max_ctx;
    a.eps = c.rms_eps; a.log2_theta = std::log2((double)c.rope_theta);
    a.token_src = token_src; a.token_stride = token_stride; a.rows_per_token = rows_per_token;
    a.ctx_len = ctx_len; a.kcache = kcache; a.vcache = vcache; a.H = H;
    a.ctl = reinterpret_cast<uint32_t*>(ctl); a.buf = buf; a.layer_bytes = L.layer; a.set_bytes = L.layer * (uint32_t)c.layers;
    static_assert(TABED_BODY_MAX_LAYERS < 256, "the key's fields");
    a.key = 1ull | ((uint64_t)rows << 1) | ((uint64_t)c.layers << 8) | ((uint64_t)c.d << 16) | ((uint64_t)c.heads << 32) | ((uint64_t)c.d_ff << 44);
    a.off_q = L.off_q; a.off_kn = L.off_kn; a.off_vn = L.off_vn; a.off_po = L.off_po; a.off_att = L.off_att; a.off_xa = L.off_xa; a.off_act = L.off_act; a.off_xm = L.off_xm;
    a.late_from = late_from < 1 ? kGangGroups : late_from;                  // (the first always comes in time)
    a.absent = absent < 1 ? kGangGroups : absent;
    a.w = w;
    // The smallest instance that has the units: one that has more asks for the last ones again, W and activations, which the chain
    // of a phase waits for (replayed in a graph, with instances for d = 768, d_ff = 3072 and wider only / now: one layer of d = 64
    // 22.5 / 20.0 us, of d = 256 22.7 / 20.7, two 36.7 / 33.0; two of d = 512, d_ff = 2048 37.6 / 35.9, all at one row).
    auto fits = [&](int units) { return c.d <= units * 256 && c.d_ff <= units * 1024; };
    if (c.d / c.heads == 64)
        return fits(1) ? launch_gang_t<8, 1, 4>(a, s) : fits(2) ? launch_gang_t<8, 2, 8>(a, s) : fits(3) ? launch_gang_t<8, 3, 12>(a, s) : launch_gang_t<8, 4, 16>(a, s);
    return fits(1) ? launch_gang_t<16, 1, 4>(a, s) : fits(2) ? launch_gang_t<16, 2, 8>(a, s) : fits(3) ? launch_gang_t<16, 3, 12>(a, s) : launch_gang_t<16, 4, 16>(a, s);
}

}  // namespace tabed
