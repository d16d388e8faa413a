// Device code shared by the vector-path kernel files: the register scan used for compaction, token loads and
// keep-masks, the hand-off constants of the one-launch kernels, and stage 1 of the low-rank part.
#pragma once
#include "device_common.h"
#include "kernels.h"

#include <type_traits>

namespace rsparse {

// Phase time stamps, only in builds with -DRSPARSE_STAMPS=1 (python -m paper_2504_19449_amd.build --stamps): every wave of
// the one-launch kernels writes one record of kStampWords 64-bit words -- {kind | workgroup << 8 | wave << 40,
// stamps of the 100 MHz wall clock at its phase boundaries (words 1..14), rows streamed (word 15)} -- into a caller's buffer
// (rsparse_debug_stamps).  Product builds compile none of it.
constexpr int kStampWords = 16;
#if RSPARSE_STAMPS
static __device__ unsigned long long *g_stamp_buf = nullptr;      // one of each per kernel file
static __device__ int g_stamp_cap = 0;
static inline hipError_t set_stamps_of_this_file(void *buf, int capacity_waves)
{
    hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(g_stamp_buf), &buf, sizeof buf);
    if (e != hipSuccess) return e;
    return hipMemcpyToSymbol(HIP_SYMBOL(g_stamp_cap), &capacity_waves, sizeof capacity_waves);
}
#define RS_STAMP_DECL unsigned long long rs_tt[kStampWords] = {}
#define RS_STAMP(i) rs_tt[i] = (unsigned long long)wall_clock64()
#define RS_STAMP_SET(i, v) rs_tt[i] = (unsigned long long)(v)
#define RS_STAMP_FLUSH(kind, wg, w)                                                                      \
    do {                                                                                                 \
        const int rs_id = (int)((blockIdx.z * gridDim.x + blockIdx.x) * (blockDim.x >> 6)) + (w);        \
        if (g_stamp_buf && (threadIdx.x & 63) == 0 && rs_id < g_stamp_cap) {                             \
            rs_tt[0] = (unsigned long long)(kind) | ((unsigned long long)(wg) << 8) | ((unsigned long long)(w) << 40); \
            for (int rs_i = 0; rs_i < kStampWords; ++rs_i) g_stamp_buf[(size_t)rs_id * kStampWords + rs_i] = rs_tt[rs_i]; \
        }                                                                                                \
    } while (0)
#else
#define RS_STAMP_DECL
#define RS_STAMP(i)
#define RS_STAMP_SET(i, v)
#define RS_STAMP_FLUSH(kind, wg, w)
#endif

namespace {

// Inclusive prefix sum of `v` over the 64 lanes of a wave (all lanes must be active), with data-parallel
// primitives: three shifted adds inside groups of four lanes, two masked row shifts that complete each row
// of 16, then the row totals are broadcast down (lane 15 into rows 1 and 3, lane 31 into rows 2 and 3).
// Lanes without a source, and lanes masked off, add zero.  Seven register-to-register steps; the same scan
// through LDS-routed shuffles measured 0.3-0.4 us per call on the path to the first weight load.
__device__ __forceinline__ int wave_inclusive_scan(int v)
{
    constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
    int x = v;
    x += __builtin_amdgcn_update_dpp(0, v, kRowShr + 1, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, v, kRowShr + 2, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, v, kRowShr + 3, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, kRowShr + 4, 0xf, 0xe, false);
    x += __builtin_amdgcn_update_dpp(0, x, kRowShr + 8, 0xf, 0xc, false);
    x += __builtin_amdgcn_update_dpp(0, x, kRowBcast15, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, kRowBcast31, 0xc, 0xf, false);
    return x;
}

// Channels [c, c+8) of the nb tokens of one batch tile, in two steps so that callers can put the
// loads of several channel groups in flight before the first compare.
template <int BT>
__device__ __forceinline__ void load_raw8(const uint16_t *X, int b0, int nb, int d_in, int c, u32x4 (&raw)[BT])
{
#pragma unroll
    for (int b = 0; b < BT; ++b)
        raw[b] = b < nb ? *reinterpret_cast<const u32x4 *>(X + (size_t)(b0 + b) * d_in + c) : u32x4{0, 0, 0, 0};
}

// The rules of the tokens of one batch tile (wave-uniform).
template <int BT>
struct TileRules {
    KeepRule r[BT];
    bool sgn;
    bool exact;          // false: plain thresholds on the magnitude (keep_threshold applies); true: the general form
    bool per_token;      // the rules differ from token to token (fixed-count activation)
};
// EXT = false: the launch is known (on the host) to use nothing but a plain threshold on the magnitude; the
// general forms then drop out at compile time.
template <int BT, bool EXT = true>
__device__ __forceinline__ void load_rules(const LayerView &L, int b0, int nb, TileRules<BT> &t)
{
    if (EXT) {
        t.sgn = L.keep_signed != 0;
        t.per_token = L.rules != nullptr;
        t.exact = t.per_token || t.sgn;
#pragma unroll
        for (int b = 0; b < BT; ++b) t.r[b] = rule_of(L, b0 + (b < nb ? b : 0));
    } else {
        t.sgn = t.per_token = t.exact = false;
#pragma unroll
        for (int b = 0; b < BT; ++b) t.r[b] = KeepRule{L.tau_ge, __builtin_nanf(""), -1, 0};
    }
}

// Per-token keep masks (bit e = channel c+e kept) of loaded channels.  With union_all
// (batch_mask_mode 1) every token's mask becomes the union over the WHOLE batch.  Returns the union
// over the tile's tokens.
template <int DT, int BT>
__device__ __forceinline__ uint32_t masks_of8(const LayerView &L, const uint16_t *X, int batch, int b0, int nb, int d_in, int c,
                                              const TileRules<BT> &rules, bool union_all, const u32x4 (&raw)[BT],
                                              uint32_t (&m)[BT])
{
    uint32_t u = 0;
    // the threshold form is the common one and sits on every workgroup's path to its first weight load (this code runs
    // once per launch, from a cold instruction cache): it keeps its own short loop; the fixed-count form is out of line
    if (__builtin_expect(!rules.exact, 1)) {
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            m[b] = 0;
            if (b < nb) {
                float xv[8];
                unpack8<DT>(raw[b], xv);
#pragma unroll
                for (int e = 0; e < 8; ++e) m[b] |= (uint32_t)keep_threshold(xv[e], rules.r[b]) << e;
            }
            u |= m[b];
        }
    } else {
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            m[b] = 0;
            if (b < nb) {
                float xv[8];
                unpack8<DT>(raw[b], xv);
#pragma unroll
                for (int e = 0; e < 8; ++e) m[b] |= (uint32_t)keep(xv[e], c + e, rules.r[b], rules.sgn) << e;
            }
            u |= m[b];
        }
    }
    if (union_all) {
        for (int bb = 0; bb < batch; ++bb) {
            if (bb >= b0 && bb < b0 + nb) continue;
            const KeepRule rr = rules.per_token ? rule_of(L, bb) : rules.r[0];
            u32x4 r2 = *reinterpret_cast<const u32x4 *>(X + (size_t)bb * d_in + c);
            float f[8];
            unpack8<DT>(r2, f);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                u |= (uint32_t)(rules.exact ? keep(f[e], c + e, rr, rules.sgn) : keep_threshold(f[e], rr)) << e;
        }
#pragma unroll
        for (int b = 0; b < BT; ++b) m[b] = (b < nb) ? u : 0u;
    }
    return u;
}

// Channel groups (of 8 channels) a thread keeps in flight while it reads the token(s).  The code that turns a
// group into keep-bits is unrolled once per group and runs once per launch, straight from a cold
// instruction cache: 3 groups (24 channels per thread and trip, 12288 channels per trip of 512 lanes) measured
// faster than 8 (14.8 vs 15.0 us per linear on the benchmark), 2 and 4 in between.
template <int BT>
struct TokenBatch { static constexpr int kGroups = BT >= 8 ? 1 : (BT == 4 ? 2 : 3); };

// t_pub entries hold this pattern until the stage-1 workgroups have written them.  No computed
// value has it: NaNs made by the ALU are canonical, and NaNs widened from 16-bit inputs have zero
// low bits; the producer maps it to the canonical NaN anyway.
constexpr uint32_t kNotReady = 0xffffffffu;
// How lowrank_rows hands t over: plain stores for a following launch, or to the launch that runs -- in the one-launch 4-bit
// kernel through entries that hold kNotReady until written (reset at the end of the launch), in the others with tags.
constexpr int kPubPlain = 0, kPubNotReady = 1, kPubTagged = 2;
// Bound on re-reads of an entry that is not ready.  The producers are workgroups with lower
// indices (dispatched before the caller), so the wait ends; the bound only turns an impossible
// schedule into an error flag instead of a hang.
constexpr long long kWaitLimitTicks = 50000000;      // 0.5 s of the 100 MHz wall clock
constexpr int kWaitLimitPolls = 1 << 20;

// Keep a wave-uniform kernel argument in scalar registers from here on.  Left alone, the compiler re-reads
// kernel arguments at their uses -- a scalar-cache round trip and a wait each time, e.g. in front of every
// single load of the token (six dependent waits before the first token load became three; the scalar cache
// hits are cheap, so this measured neutral on the benchmark).
__device__ __forceinline__ int pin(int v) { __asm__ volatile("" : "+s"(v)); return v; }
__device__ __forceinline__ float pin(float v) { __asm__ volatile("" : "+s"(v)); return v; }
template <typename T>
__device__ __forceinline__ const T *pin(const T *p)
{
    uintptr_t u = reinterpret_cast<uintptr_t>(p);
    __asm__ volatile("" : "+s"(u));
    // back through a global-memory pointer type, so that loads stay global loads (not generic ones)
    typedef const T __attribute__((address_space(1))) *global_ptr;
    return (const T *)reinterpret_cast<global_ptr>(u);
}

// A pointer the compiler has lost track of (out of inline asm) as one into global memory: global, not generic accesses.
template <typename T>
__device__ __forceinline__ T *as_global(T *p)
{
    typedef T __attribute__((address_space(1))) *global_ptr;
    return (T *)reinterpret_cast<global_ptr>(reinterpret_cast<uintptr_t>(p));
}

// Balanced share [lo, hi) of n items for part p of `parts`: the first n % parts shares hold one item more.
// 32-bit arithmetic on wave-uniform values -- a 64-bit division is some 200 emulated instructions here,
// and it sat on every workgroup's path to its first weight load.
__device__ __forceinline__ void balanced_share(int n, int parts, int p, int &lo, int &hi)
{
    const unsigned un = (unsigned)uniform(n), up = (unsigned)uniform(parts), pp = (unsigned)uniform(p);
    const unsigned base = un / up, rem = un - base * up;
    lo = (int)(pp * base + min(pp, rem));
    hi = lo + (int)base + (pp < rem ? 1 : 0);
}

// Tagged hand-off of t inside one launch.  Entries are {tag, fp32 bits}; a launch's tag is one more than its generation, a
// number that is kept per column tile (strip) for those who read t and per batch tile for those who write it, each in the line
// of the arrival counter that ends its use: whoever arrives last puts the counter back and bumps the generation.  All of them
// move once per launch and start at zero together, so they agree.  Nobody can read a generation after its bump (everybody
// who reads it arrives afterwards), entries of earlier launches never match, and nothing has to be reset at the end of a
// launch: a reset needs to know that every tile has read t, which is one more counter between the sums and the stores (0.6 us).
__device__ __forceinline__ uint32_t generation(const int *line)
{
    return (uint32_t)__hip_atomic_load(line + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void end_of_line(int *line)
{
    __hip_atomic_store(line, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(line + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish_t(unsigned long long *entry, uint32_t gen, float v)
{
    __hip_atomic_store(entry, ((unsigned long long)(gen + 1u) << 32) | as_u(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Token slots that a call does not use keep the tags of earlier launches.  Every 2^30 launches they are written too, so that
// none is ever old enough to match again: slots bt .. of batch tile 0 (the others are always full) of rank index `row`.
__device__ __forceinline__ void refresh_unused(unsigned long long *t_tag, int rank, int t_slots, int bt, int z, uint32_t gen, int row)
{
    if (z == 0 && (gen & 0x3fffffffu) == 0u)
        for (int sl = bt; sl < min(kMaxBT, t_slots); ++sl) publish_t(t_tag + (size_t)sl * rank + row, gen, 0.f);
}

// Sum over the 64 lanes, in lane 63: rotations inside the rows of 16 lanes, then the row totals broadcast down.
__device__ __forceinline__ float wave_sum63(float v)
{
    constexpr int kRowRor = 0x120, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
    auto dpp = [](float x, auto ctrl, auto rows) { return as_f((uint32_t)__builtin_amdgcn_update_dpp(0, (int)as_u(x), decltype(ctrl)::value, decltype(rows)::value, 0xf, false)); };
    v += dpp(v, std::integral_constant<int, kRowRor + 8>{}, std::integral_constant<int, 0xf>{});
    v += dpp(v, std::integral_constant<int, kRowRor + 4>{}, std::integral_constant<int, 0xf>{});
    v += dpp(v, std::integral_constant<int, kRowRor + 2>{}, std::integral_constant<int, 0xf>{});
    v += dpp(v, std::integral_constant<int, kRowRor + 1>{}, std::integral_constant<int, 0xf>{});
    v += dpp(v, std::integral_constant<int, kRowBcast15>{}, std::integral_constant<int, 0xa>{});
    v += dpp(v, std::integral_constant<int, kRowBcast31>{}, std::integral_constant<int, 0xc>{});
    return v;
}

// Raw buffer descriptors: an access past the end reads zero without touching memory, so that loads can be unconditional.
constexpr int kBufferFlags = 0x00020000;               // raw buffer, 32-bit elements
constexpr uint32_t kOutside = 0x80000000u;             // past any descriptor used here
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const uint16_t *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p), 0, (int)bytes, kBufferFlags);
}
template <bool NT>
__device__ __forceinline__ u32x4 buffer_load16(__amdgpu_buffer_rsrc_t rsrc, uint32_t off)
{
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, NT ? 2 : 0));
}

// ---------------------------------------------------------------------------------------------
// Stage 1 of the low-rank part inside a one-launch kernel: t_i = sum_c (S_r V_r^T)[i, c] (x - sigma_t(x))_c.
// Everything else in the launch ends with rows that need t, so this is a chain of latencies first: a workgroup takes `rows`
// rows of S_r V_r^T, its waves share the channels (wave w every nw-th run of 512), and a lane requests its 8 channels of the
// token(s) and of S1Shape::kRows rows at once -- the rows do not depend on the token --, masks the token in registers (once for all
// rows) and multiplies; the waves meet in LDS and one lane per row and token publishes.  No staging of the token and no barrier
// before the last product.  (A wave per row over a token staged in LDS published t 1.5 us later at 4096 channels.)
// ---------------------------------------------------------------------------------------------
struct Stage1Args {
    const uint16_t *X, *SVt;
    int *sync;
    unsigned long long *t_tag;
    int d_in, rank, batch, rows;       // rows: of S_r V_r^T per workgroup
    int wgs, t_slots, union_all, skip; // workgroups; token slots of t_tag; test hook: publish nothing
    float tau_ge;
    int waves;
    int chunk;                         // lowrank_rows: channels of the token(s) in LDS at once; 0: stage1_rows
};
inline Stage1Args stage1_args(const LayerView &L, const void *X, int batch, const Launch &cfg, int wgs, int waves, int chunk)
{
    return Stage1Args{(const uint16_t *)X, L.SVt, L.sync, L.t_tag, L.d_in, L.rank, batch, cfg.lowrank_rows, wgs, L.t_slots,
                      L.batch_mask_mode == 1, cfg.skip_stage1, L.tau_ge, waves, chunk};
}
template <int BT> struct S1Shape {
    static constexpr int kRows = BT >= 4 ? 2 : 4;      // rows that share a token in registers
};

template <int DT, int BT, bool EXT>
__device__ __forceinline__ void stage1_rows(const Stage1Args &args, const LayerView &L, unsigned char *smem, int wg, int z)
{
    constexpr int RW = S1Shape<BT>::kRows;
    Stage1Args s = args;
    __asm__ volatile("" : "+s"(s.X), "+s"(s.SVt), "+s"(s.sync), "+s"(s.t_tag), "+s"(s.d_in), "+s"(s.rank), "+s"(s.batch), "+s"(s.rows), "+s"(s.wgs),
                     "+s"(s.union_all), "+s"(s.tau_ge), "+s"(s.waves));
    const int tid = threadIdx.x, lane = tid & 63, w = uniform(tid >> 6), nw = s.waves;
    const int d_in = s.d_in, r = s.rank, b0 = z * BT, nb = min(BT, s.batch - b0);
    int *const line = as_global(s.sync) + kSyncStage1 + z * kSyncLine;
    float *const s_part = reinterpret_cast<float *>(smem);                  // [2][RW * BT][nw]
    const __amdgpu_buffer_rsrc_t tokens = buffer_of(s.X, (uint32_t)s.batch * d_in * 2u);
    RS_STAMP_DECL;
    RS_STAMP(1);
    uint32_t gen = 0;
    TileRules<BT> rules;
    load_rules<BT, EXT>(L, b0, nb, rules);
    if (!EXT) {
#pragma unroll
        for (int b = 0; b < BT; ++b) rules.r[b].ge = s.tau_ge;
    }
    const int row_end = min(r, (wg + 1) * s.rows);
    // (rows, run of 512 channels) in the order in which they are taken: two are in flight, also from one set of rows to the next
    struct Pos { int row0, c0; };
    auto advance = [&](Pos &p) {
        p.c0 += nw * 512;
        if (p.c0 - w * 512 >= d_in) { p.c0 = w * 512; p.row0 += RW; }
    };
    float part[RW][BT];
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int b = 0; b < BT; ++b) part[i][b] = 0.f;
    struct Run { u32x4 x[BT], v[RW]; };
    auto request = [&](const Pos &p, Run &q) {
        const int c = p.c0 + lane * 8, n_rows = max(0, min(RW, row_end - p.row0));     // (past the workgroup's rows: outside)
        const __amdgpu_buffer_rsrc_t rows = buffer_of(s.SVt + (size_t)min(p.row0, r - 1) * d_in, (uint32_t)n_rows * d_in * 2u);
#pragma unroll
        for (int b = 0; b < BT; ++b) q.x[b] = buffer_load16<false>(tokens, c < d_in && b < nb ? (uint32_t)((b0 + b) * d_in + c) * 2u : kOutside);
#pragma unroll
        for (int i = 0; i < RW; ++i) q.v[i] = buffer_load16<true>(rows, c < d_in ? (uint32_t)(i * d_in + c) * 2u : kOutside);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto use = [&](const Pos &p, const Run &q) {
        const int c = p.c0 + lane * 8;
        float xf[BT][8];
#pragma unroll
        for (int b = 0; b < BT; ++b) unpack8<DT>(q.x[b], xf[b]);
        uint32_t other_kept = 0u;
        if (BT > 1 && s.union_all) {
            // every token uses the union over the WHOLE batch (also the tokens of other batch tiles)
            for (int bb = 0; bb < s.batch; ++bb) {
                if (bb >= b0 && bb < b0 + nb) continue;
                float of[8];
                unpack8<DT>(buffer_load16<false>(tokens, c < d_in ? (uint32_t)(bb * d_in + c) * 2u : kOutside), of);
#pragma unroll
                for (int e = 0; e < 8; ++e) other_kept |= (uint32_t)keep(of[e], c + e, EXT ? rule_of(L, bb) : rules.r[0], rules.sgn) << e;
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            bool kept[BT], any = ((other_kept >> e) & 1u) != 0u;
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                kept[b] = EXT ? keep(xf[b][e], c + e, rules.r[b], rules.sgn) : keep_threshold(xf[b][e], rules.r[b]);
                any = any || (kept[b] && b < nb);
            }
#pragma unroll
            for (int b = 0; b < BT; ++b) xf[b][e] = (BT > 1 && s.union_all ? any : kept[b]) ? 0.f : xf[b][e];
        }
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            float f[8];
            unpack8<DT>(q.v[i], f);
#pragma unroll
            for (int b = 0; b < BT; ++b)
#pragma unroll
                for (int e = 0; e < 8; ++e) part[i][b] = __builtin_fmaf(f[e], xf[b][e], part[i][b]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // the last run of a set of rows: the waves meet in LDS (two buffers in turn: a wave is never two sets ahead of another)
    int buffer = 0;
    auto finish = [&](const Pos &p) {
        float *const sum = s_part + buffer * (RW * BT * nw);
        buffer ^= 1;
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                const float v = wave_sum63(part[i][b]);
                if (lane == 63) sum[(i * BT + b) * nw + w] = v;
                part[i][b] = 0.f;
            }
        __syncthreads();
        const int i = tid / BT, b = tid % BT;
        if (tid < RW * BT && p.row0 + i < row_end && !s.skip) {
            float v = 0.f;
            for (int k = 0; k < nw; ++k) v += sum[tid * nw + k];
            publish_t(as_global(s.t_tag) + ((size_t)z * BT + b) * r + p.row0 + i, gen, v);
            if (b == 0) refresh_unused(as_global(s.t_tag), r, s.t_slots, BT, z, gen, p.row0 + i);
        }
    };
    auto last_run = [&](const Pos &p) { return p.row0 < row_end && p.c0 - w * 512 + nw * 512 >= d_in; };
    Run qa, qb;
    Pos ahead{wg * s.rows, w * 512}, at = ahead;
    request(ahead, qa);
    advance(ahead);
    gen = generation(line);
    while (at.row0 < row_end) {
        request(ahead, qb);
        advance(ahead);
        use(at, qa);
        RS_STAMP(2);
        if (last_run(at)) finish(at);
        advance(at);
        request(ahead, qa);
        advance(ahead);
        use(at, qb);
        if (last_run(at)) finish(at);
        advance(at);
    }
    RS_STAMP(3);
    RS_STAMP(4);
    static_assert(RW * BT <= 64, "the lanes that use the generation are wave 0's");
    if (tid == 0 && __hip_atomic_fetch_add(line, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == s.wgs - 1) end_of_line(line);
    RS_STAMP(5);
    RS_STAMP_FLUSH(1, wg, w);
}

// ---------------------------------------------------------------------------------------------
// Stage 1 of the low-rank part (Sec. 3.4): t_i = sum_c (S_r V_r^T)[i, c] * (x - sigma_t(x))_c.
// A workgroup stages the masked token(s) in LDS (kept channels zeroed); each of its waves then dots
// whole rows of S_r V_r^T against them, eight 16-byte loads in flight per lane.  A row is complete
// inside one wave, so t needs no cross-workgroup sum, no atomics and no zeroing.
// t is stored [batch tile][token][rank].  At most kRowsPerWave rows per wave (host-enforced).
// ---------------------------------------------------------------------------------------------
constexpr int kRowsPerWave = 4;

struct RowsArgs {
    const uint16_t *X;
    int batch, rows, chunk, skip, wgs, t_slots;      // (as in Stage1Args)
};

template <int DT, int BT, int PUB, bool EXT = true>
__device__ __forceinline__ void lowrank_rows(const RowsArgs &a, const LayerView &L, unsigned char *smem, int wg, int z)
{
    // loads per batch and lane, batches in flight: two batches of six for one token; more tokens keep more of the
    // register file for the token values, and a second batch then spills
    constexpr int LU = BT == 1 ? 6 : 8, kRowBatches = BT == 1 ? 2 : 1;
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, w = tid >> 6, nw = nthr >> 6;
    const int d_in = L.d_in, r = L.rank;
    const int b0 = z * BT;
    const int nb = min(BT, a.batch - b0);
    const bool union_all = L.batch_mask_mode == 1;
    int *const line = L.sync + kSyncStage1 + z * kSyncLine;
    uint32_t gen = 0;
    if constexpr (PUB == kPubTagged) gen = generation(line);
    TileRules<BT> rules;
    load_rules<BT, EXT>(L, b0, nb, rules);
    uint16_t *s_xm = reinterpret_cast<uint16_t *>(smem);                           // [BT][chunk]
    const int row_lo = wg * a.rows, row_hi = min(r, row_lo + a.rows);

    float part[kRowsPerWave][BT];
#pragma unroll
    for (int sl = 0; sl < kRowsPerWave; ++sl)
#pragma unroll
        for (int b = 0; b < BT; ++b) part[sl][b] = 0.f;

    for (int c0 = 0; c0 < d_in; c0 += a.chunk) {
        const int len = min(a.chunk, d_in - c0);
        const int nq = len / 8;
        if (c0 > 0) __syncthreads();
        constexpr int PB = TokenBatch<BT>::kGroups;
        for (int q0 = tid; q0 < nq; q0 += nthr * PB) {
            u32x4 raw[PB][BT];
#pragma unroll
            for (int p = 0; p < PB; ++p)
                if (q0 + p * nthr < nq) load_raw8<BT>(a.X, b0, nb, d_in, c0 + (q0 + p * nthr) * 8, raw[p]);
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                const int q = q0 + p * nthr;
                if (q < nq) {
                    uint32_t m[BT];
                    masks_of8<DT, BT>(L, a.X, a.batch, b0, nb, d_in, c0 + q * 8, rules, union_all, raw[p], m);
#pragma unroll
                    for (int b = 0; b < BT; ++b) {
                        u32x4 o = raw[p][b];
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if ((m[b] >> e) & 1u) o[e >> 1] &= (e & 1) ? 0x0000ffffu : 0xffff0000u;   // kept -> 0
                        *reinterpret_cast<u32x4 *>(s_xm + (size_t)b * a.chunk + q * 8) = o;
                    }
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int sl = 0; sl < kRowsPerWave; ++sl) {
            const int i = row_lo + w + sl * nw;
            if (i < row_hi) {
                const uint16_t *row = L.SVt + (size_t)i * d_in + c0;
                if constexpr (kRowBatches == 1) {
                    for (int q0 = lane; q0 < nq; q0 += 64 * LU) {
                        u32x4 v[LU];
#pragma unroll
                        for (int u = 0; u < LU; ++u) {
                            const int q = q0 + u * 64;
                            v[u] = (q < nq) ? ldg16<true>(row + q * 8) : u32x4{0, 0, 0, 0};       // streamed once
                        }
#pragma unroll
                        for (int u = 0; u < LU; ++u) {
                            const int q = q0 + u * 64;
                            if (q < nq) {
                                float f[8];
                                unpack8<DT>(v[u], f);
#pragma unroll
                                for (int b = 0; b < BT; ++b) {
                                    float xf[8];
                                    unpack8<DT>(*reinterpret_cast<const u32x4 *>(s_xm + (size_t)b * a.chunk + q * 8), xf);
#pragma unroll
                                    for (int e = 0; e < 8; ++e) part[sl][b] = __builtin_fmaf(f[e], xf[e], part[sl][b]);
                                }
                            }
                        }
                    }
                } else {
                // kRowBatches batches of LU loads in flight per lane; unconditional loads (positions past the row's
                // end re-read its last piece and are dropped) so that the compiler counts the outstanding ones
                // exactly -- with one batch at a time a wave needed one dependent round trip per 8 KiB of its row
                // (seven for a 28672-channel down projection) through a saturated memory system
                u32x4 v[kRowBatches][LU];
                const int q_last = nq - 1;
                constexpr int kStep = 64 * LU;
                auto request = [&](u32x4 (&dst)[LU], int q0) {
#pragma unroll
                    for (int u = 0; u < LU; ++u) dst[u] = ldg16<true>(row + min(q0 + u * 64, q_last) * 8);      // streamed once
                };
                int q0 = lane;
#pragma unroll
                for (int j = 0; j < kRowBatches; ++j)
                    if (j * kStep < nq) request(v[j], q0 + j * kStep);
                bool more = nq > 0;                      // wave-uniform
                while (more) {
#pragma unroll
                    for (int j = 0; j < kRowBatches; ++j) {
                        if (more) {
#pragma unroll
                            for (int u = 0; u < LU; ++u) {
                                const int q = q0 + u * 64;
                                if (q < nq) {
                                    float f[8];
                                    unpack8<DT>(v[j][u], f);
#pragma unroll
                                    for (int b = 0; b < BT; ++b) {
                                        float xf[8];
                                        unpack8<DT>(*reinterpret_cast<const u32x4 *>(s_xm + (size_t)b * a.chunk + q * 8), xf);
#pragma unroll
                                        for (int e = 0; e < 8; ++e) part[sl][b] = __builtin_fmaf(f[e], xf[e], part[sl][b]);
                                    }
                                }
                            }
                            const int qn = q0 + kRowBatches * kStep;
                            if (qn - lane < nq) request(v[j], qn);
                            q0 += kStep;
                            more = q0 - lane < nq;
                        }
                    }
                }
                }
            }
        }
    }
#pragma unroll
    for (int sl = 0; sl < kRowsPerWave; ++sl) {
        const int i = row_lo + w + sl * nw;
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            const float v = wave_sum(part[sl][b]);
            if (lane == 0 && i < row_hi) {
                const size_t at = ((size_t)z * BT + b) * r + i;
                if (PUB == kPubTagged) {
                    if (!a.skip) publish_t(L.t_tag + at, gen, v);
                } else if (PUB == kPubNotReady) {
                    if (a.skip) continue;
                    uint32_t bits = as_u(v);
                    if (bits == kNotReady) bits = 0x7fc00000u;
                    __hip_atomic_store(L.t_pub + at, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    L.t[at] = v;
                }
            }
        }
        if (PUB == kPubTagged && lane == 0 && i < row_hi && !a.skip) refresh_unused(L.t_tag, r, a.t_slots, BT, z, gen, i);
    }
    if constexpr (PUB == kPubTagged) {
        __syncthreads();                       // every wave has used the generation
        if (tid == 0 && __hip_atomic_fetch_add(line, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.wgs - 1) end_of_line(line);
    }
}

// Stage 1 of a one-launch kernel of 16-bit weights, in the form that the host chose (stage1_chunk).
template <int DT, int BT, bool EXT>
__device__ __forceinline__ void stage1_tagged(const Stage1Args &s, const LayerView &L, unsigned char *smem, int wg, int z)
{
    if constexpr (BT >= 4) {
        if (BT >= 8 || s.chunk > 0) {
            lowrank_rows<DT, BT, kPubTagged, EXT>(RowsArgs{s.X, s.batch, s.rows, s.chunk, s.skip, s.wgs, s.t_slots}, L, smem, wg, z);
            return;
        }
    }
    if constexpr (BT < 8) stage1_rows<DT, BT, EXT>(s, L, smem, wg, z);
}

}  // namespace
}  // namespace rsparse
