// gfx950 matrix-core path of the R-Sparse linear layer (R-Sparse, Sec. 3.4) for 5 to 32 tokens, and of the dense product
// for 1 to 32, over a copy of W in operand layout (dense_rowmajor = 1).
//
// At 5 tokens and more the union of kept channels is nearly all of them and 2*B flops per weight byte is more than the
// vector ALU sustains at HBM speed, so all three products are skinny GEMMs on MFMA, still one pass over the weights:
//
//   Y_s = (X (.) m)  W^T            rows of W   [d_out][d_in] row-major  (dense, per-token masks in X)
//   t   = (X (.) !m) (S_r V_r^T)^T  rows of SVt [r][d_in]
//   Y   = round(Y_s + t U_r^T)      rows of U   [d_out][r]
//
// Operands of v_mfma_f32_16x16x32_{bf16,f16}: lane l supplies 8 consecutive k
// (one 16-byte load) of row l%16 at k-group l/16.  A = 16 weight rows x 32 k, B = 32 k x 16
// tokens, D[row][token] fp32: lane l, register j holds row 4*(l/16)+j, token l%16.
//
// ONE launch per call (a group of layers that read the same input shares it).  The matrices are kept in that operand
// layout (MatrixView), so that a wave's load is 1 KiB of consecutive bytes; from row-major rows it is 16 pieces of
// 64 bytes a row pitch apart, which the first-level cache drops half-used (8192 x 8192, 32 tokens: 74 us against 51).
// A unit is 16 * NB rows of W over the WHOLE contraction, owned by one workgroup whose waves take its batches of loads in
// turn: no sum of outputs crosses workgroups, so there are no atomics on outputs, no accumulators in memory, no second
// launch.  Bound by HBM: the tokens come from L2, change to the operand layout through the wave's own LDS and are masked
// there in their 16-bit patterns (five packed integer operations per two values); the waves' D tiles meet in LDS once.
// The first workgroups of the grid take t, a (block of 16 rank indices, K slice) each, and wait for nothing; the last
// slice of a block splits the sums into two 16-bit halves (hi + lo, ~16 mantissa bits of the fp32 t) and stores them in
// operand layout with write-through stores, waits for these to be acknowledged and sets the block's flag.  A unit of W
// waits for the flags (bounded) when its rows are done and adds U_r t.  The t buffer is read with ordinary loads: its
// lines are first touched in a launch by readers that have seen the flags, so no older copy of them is in a cache.
// Measured (us per call, before: a first launch with sums over K slices in fp32 atomics, a split launch and a finish
// launch): 8192 x 8192 r 1024 60.3 -> 41.7 at 32 tokens, 53.1 -> 34.7 at 8; 4096 x 4096 r 256 23.1 -> 14.6 at 8; dense
// 4096 -> 14336 (two) and back 93.1 -> 71.1 at 16.
#include "kernels.h"
#include "device_common.h"
#include "device_stage1.h"

#include <algorithm>

namespace rsparse {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

constexpr int kMfmaK = 32;        // contraction depth of one MFMA
// MFMA steps of one batch of loads, for units of NB blocks.  Measured on plain streams of this shape (512 workgroups of
// 8 waves, 134 MB): two batches of 4 KiB per wave in flight 6.3 TB/s, of 8 KiB 5.6, of 16 KiB 4.5 -- more requests than
// the memory system takes only push each other out.
template <int NB> struct StepsOf { static constexpr int value = NB == 1 ? 4 : 2; };

template <int DT>
__device__ __forceinline__ f32x4 mfma16(const u32x4 a, const u32x4 b, const f32x4 c)
{
    if (DT == BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

template <int DT>
__device__ __forceinline__ uint16_t narrow(float f) { return DT == F16 ? to_f16(f) : to_bf16(f); }

// The lo half of t is stored scaled by a power of two (exact): in fp16 the remainder t - hi would otherwise fall into
// the subnormals for |t| below ~0.1 and lose the bits it is there to keep.
template <int DT> struct LoScale { static constexpr float value = DT == F16 ? 2048.0f : 1.0f; };

// ---------------------------------------------------------------------------------------------
// The sparsification function on packed 16-bit patterns.  Magnitudes order like their patterns, so |x| >= t is
// pattern(|x|) >= pattern_min (host-computed, exact), signed thresholds compare the sign-magnitude pattern as a two's
// complement number, and NaN patterns lie above infinity's.
// ---------------------------------------------------------------------------------------------
struct KeepPattern {
    uint32_t min2, inf2;       // smallest kept pattern and infinity's, each twice
};

// 0xffff in every half of x that the token DROPS.
template <bool SIGNED>
__device__ __forceinline__ uint32_t dropped2(uint32_t x, const KeepPattern &kp)
{
    const s16x2 mag = __builtin_bit_cast(s16x2, x & 0x7fff7fffu);
    s16x2 key = mag;
    if (SIGNED) {
        const s16x2 sgn = __builtin_bit_cast(s16x2, x) >> 15;
        key = (mag ^ sgn) - sgn;
    }
    const s16x2 below = __builtin_elementwise_sub_sat(key, __builtin_bit_cast(s16x2, kp.min2));
    const s16x2 nan = __builtin_bit_cast(s16x2, kp.inf2) - mag;
    return __builtin_bit_cast(uint32_t, (s16x2)((below | nan) >> 15));
}

__device__ __forceinline__ uint32_t and_over_16_lanes(uint32_t v)
{
    constexpr int kRowRor = 0x120;
    v &= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowRor + 8, 0xf, 0xf, false);
    v &= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowRor + 4, 0xf, 0xf, false);
    v &= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowRor + 2, 0xf, 0xf, false);
    v &= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kRowRor + 1, 0xf, 0xf, false);
    return v;
}

// All of this wave's earlier atomics and stores have been performed.
__device__ __forceinline__ void wait_own_writes()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
}

constexpr int kMaskNone = 0, kMaskOwn = 1, kMaskUnion = 2;   // MfmaJob::mask_mode
constexpr int kMaskSigned = 4;                               // ... + the rule applies to x itself

// The part of the tokens a unit works on: kept values (want = 0) or dropped ones (want = ~0), the others zeroed.
// Frags of one step: NF token tiles of 16; with the union mask a channel counts as kept if any token keeps it (lanes
// past the batch hold a copy of its last token).
template <int NF, int MODE>
__device__ __forceinline__ void mask_step(u32x4 (&b)[NF], const KeepPattern &kp, uint32_t want)
{
    if (MODE == kMaskNone) return;
    uint32_t d[NF][4];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 4; ++i) d[f][i] = dropped2<(MODE & kMaskSigned) != 0>(b[f][i], kp);
    if (MODE & kMaskUnion) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t all = d[0][i];
#pragma unroll
            for (int f = 1; f < NF; ++f) all &= d[f][i];
            all = and_over_16_lanes(all);
#pragma unroll
            for (int f = 0; f < NF; ++f) d[f][i] = all;
        }
    }
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int i = 0; i < 4; ++i) b[f][i] &= ~(d[f][i] ^ want);
}

struct MfmaJob {
    const uint16_t *W, *SVt, *U; // operand layout (MatrixView)
    unsigned char *t;            // t in operand layout: [step of 32 rank indices][token tile][hi, lo][64 lanes][16 bytes]
    float *t_acc;                // [block of 16 rank indices][token tile][4][64] fp32 sums of t's K slices, zero between calls
    int *t_flags;                // a flag per block of t, zero between calls; then an arrival counter per block
    void *Y;
    const float *bias;
    uint32_t *chan_bits;         // [d_in] bit b = token b keeps the channel (read-back), or nullptr
    int *sync;
    int d_out, rank;
    int out_dtype, mask_mode;
    KeepPattern kp;
    int t_blocks, w_units;       // blocks of S_r V_r^T (0: no low-rank part), units of W
};
struct MfmaArgs {
    MfmaJob job[kMaxGroupLayers];
    int t_end[kMaxGroupLayers];  // t tasks (block, K slice) of jobs 0..i
    int w_end[kMaxGroupLayers];  // units of W of jobs 0..i
    const uint16_t *X;
    int n, batch, d_in, t_slices;
    int phases;                  // 1: t, 2: the units of W, 3: both in this launch (the units of W wait for t)
    int wait_polls, skip_stage1;
};

// One batch of a wave: S steps of NB weight tiles (1 KiB each) and the same 32 * S channels of all tokens, 4 * S lanes to
// a token.
template <int NB, int NF>
struct Batch {
    static constexpr int S = StepsOf<NB>::value, K = kMfmaK * S, kLanes = 4 * S, kX = NF * S;
    static constexpr int kPitch = K * 2 + 16;   // bytes of a token in LDS: the 16 tokens of a read hit 16 bank groups
    u32x4 a[S][NB], x[kX];
};

// Weights are read once: non-temporal (8192 x 8192 at 32 tokens 51.7 against 54.7 us with ordinary loads).
__device__ __forceinline__ u32x4 ld16(const unsigned char *p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
}

// Batch `bi` of the contraction (past its end: its last values again).
template <int NB, int NF>
__device__ __forceinline__ void load_batch(const unsigned char *__restrict__ mat, const size_t (&aoff)[NB], const unsigned char *__restrict__ x,
                                           const uint32_t (&xoff)[Batch<NB, NF>::kX], int lane, int d_in, int steps, int bi,
                                           Batch<NB, NF> &v)
{
    using B = Batch<NB, NF>;
    const uint32_t k = (uint32_t)min(bi * B::K + lane % B::kLanes * 8, d_in - 8) * 2u;
#pragma unroll
    for (int j = 0; j < B::kX; ++j) v.x[j] = *reinterpret_cast<const u32x4 *>(x + (size_t)(xoff[j] + k));
#pragma unroll
    for (int u = 0; u < B::S; ++u) {
        const int s = min(bi * B::S + u, steps - 1);
#pragma unroll
        for (int i = 0; i < NB; ++i) v.a[u][i] = ld16(mat + aoff[i] + (size_t)s * 1024 + lane * 16);
    }
    __builtin_amdgcn_sched_barrier(0);      // all of them are issued here, ahead of the batch that is used next
}

template <int DT, int NB, int NF, int MODE>
__device__ __forceinline__ void use_batch(Batch<NB, NF> &v, unsigned char *sx, const KeepPattern &kp, uint32_t want, int lane,
                                          int k_end, int bi, f32x4 (&acc)[NB][NF])
{
    using B = Batch<NB, NF>;
    // the tokens change from kLanes lanes a token to the operand layout through this wave's own LDS
    const bool in = bi * B::K + lane % B::kLanes * 8 < k_end;
#pragma unroll
    for (int j = 0; j < B::kX; ++j)
        *reinterpret_cast<u32x4 *>(sx + (j * (64 / B::kLanes) + lane / B::kLanes) * B::kPitch + lane % B::kLanes * 16) =
            in ? v.x[j] : u32x4{0, 0, 0, 0};
    __builtin_amdgcn_wave_barrier();
    f32x4 sum[NB][NF];
#pragma unroll
    for (int u = 0; u < B::S; ++u) {
        u32x4 b[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f)
            b[f] = *reinterpret_cast<const u32x4 *>(sx + (f * 16 + (lane & 15)) * B::kPitch + u * 64 + (lane >> 4) * 16);
        mask_step<NF, MODE>(b, kp, want);
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int f = 0; f < NF; ++f) sum[i][f] = mfma16<DT>(v.a[u][i], b[f], u ? sum[i][f] : f32x4{0.f, 0.f, 0.f, 0.f});
    }
    // a batch's sums are added to the task's with the vector ALU: the matrix cores' own long chains of sums lose bits
    // (28672 channels: 3.8e-7 from the 64-bit result in one chain)
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[i][f] += sum[i][f];
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// A wave's batches bi, bi + nw, ... below `end`, two in flight: every load is unconditional (past the end it re-reads the
// last values, against tokens of zeros), so that the compiler counts the outstanding ones exactly and waits for the
// current batch alone.  The first batch is in va already.
template <int DT, int NB, int NF, int MODE>
__device__ __forceinline__ void stream_rows(const unsigned char *__restrict__ mat, const size_t (&aoff)[NB],
                                            const unsigned char *__restrict__ x, const uint32_t (&xoff)[Batch<NB, NF>::kX], unsigned char *sx,
                                            const KeepPattern &kp, uint32_t want, int lane, int d_in, int bi, int end, int nw,
                                            Batch<NB, NF> &va, f32x4 (&acc)[NB][NF])
{
    const int steps = (d_in + kMfmaK - 1) / kMfmaK;
    Batch<NB, NF> vb;
    const int k_end = min(end * Batch<NB, NF>::K, d_in);
    for (; bi < end; bi += 2 * nw) {
        load_batch<NB, NF>(mat, aoff, x, xoff, lane, d_in, steps, bi + nw, vb);
        use_batch<DT, NB, NF, MODE>(va, sx, kp, want, lane, k_end, bi, acc);
        load_batch<NB, NF>(mat, aoff, x, xoff, lane, d_in, steps, bi + 2 * nw, va);
        use_batch<DT, NB, NF, MODE>(vb, sx, kp, want, lane, k_end, bi + nw, acc);
    }
}

template <int DT, int NB, int NF>
__global__ __launch_bounds__(512, NF == 1 ? 4 : 2) void k_mfma_rows(const MfmaArgs ga)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, w = uniform(tid >> 6), nw = uniform(nthr >> 6);
    const int d_in = ga.d_in, batch = ga.batch;
    using B = Batch<NB, NF>;
    const int steps = (d_in + kMfmaK - 1) / kMfmaK, n_batches = (steps + B::S - 1) / B::S;
    const size_t block_bytes = (size_t)steps * 1024;
    const unsigned char *x = reinterpret_cast<const unsigned char *>(ga.X);
    // tokens past the batch repeat its last one; their results are not used
    uint32_t xoff[B::kX];
#pragma unroll
    for (int j = 0; j < B::kX; ++j) xoff[j] = (uint32_t)min(j * (64 / B::kLanes) + lane / B::kLanes, batch - 1) * (uint32_t)d_in * 2u;
    constexpr int kTiles = NB * NF;
    // a wave's LDS: its tokens' staging, and its D tiles when the waves meet
    constexpr int kWaveLds = NF * 16 * B::kPitch > kTiles * 1024 ? NF * 16 * B::kPitch : kTiles * 1024;
    unsigned char *sx = smem + (size_t)w * kWaveLds;

    // the first t_wgs workgroups take a (block, K slice) of t each and wait for nothing; the others a unit of W each
    const int t_wgs = ga.t_end[kMaxGroupLayers - 1] * (ga.phases & 1);
    const bool is_t = (int)blockIdx.x < t_wgs;
    const int first = is_t ? (int)blockIdx.x : (int)blockIdx.x - t_wgs;
    int job = 0, begin = 0;
#pragma unroll
    for (int j = 0; j < kMaxGroupLayers - 1; ++j) {
        const int e = is_t ? ga.t_end[j] : ga.w_end[j];
        if (first >= e) { job = j + 1; begin = e; }
    }
    const MfmaJob &jb = ga.job[job];
    const KeepPattern kp = jb.kp;
    const int t_slices = ga.t_slices, slice = is_t ? (first - begin) % t_slices : 0;
    const int unit = is_t ? (first - begin) / t_slices : first - begin;
    const int lo = is_t ? (int)((unsigned)(n_batches * slice) / (unsigned)t_slices) : 0;
    const int hi = is_t ? (int)((unsigned)(n_batches * (slice + 1)) / (unsigned)t_slices) : n_batches;
    const int block0 = is_t ? unit : unit * NB, n_blocks = (jb.d_out + 15) / 16;
    const unsigned char *mat = reinterpret_cast<const unsigned char *>(is_t ? jb.SVt : jb.W) + (size_t)block0 * block_bytes;
    size_t aoff[NB];                                            // (blocks past the matrix: the last one again)
#pragma unroll
    for (int k = 0; k < NB; ++k) aoff[k] = is_t ? 0 : (size_t)min(k, n_blocks - 1 - block0) * block_bytes;

    Batch<NB, NF> va;
    load_batch<NB, NF>(mat, aoff, x, xoff, lane, d_in, steps, lo + w, va);

    // ---- which tokens keep a channel, for read-back: the last wave, 16 channels at a time (a lane = a token)
    if (!is_t && w == nw - 1) {
        for (int j = 0; j < ga.n; ++j) {
            const MfmaJob &pj = ga.job[j];
            if (!pj.chan_bits) continue;
            const KeepPattern pk = pj.kp;
            const bool sgn = (pj.mask_mode & kMaskSigned) != 0;
            for (int c0 = first * 16; c0 < d_in; c0 += ((int)gridDim.x - t_wgs) * 16) {
                const int c = c0 + (lane >> 5) * 8, tok = lane & 31;
                u32x4 v = u32x4{0, 0, 0, 0};
                const bool in = c < d_in && tok < batch;
                if (in) v = *reinterpret_cast<const u32x4 *>(ga.X + (size_t)tok * d_in + c);
                const uint32_t all_tokens = batch >= 32 ? 0xffffffffu : (1u << batch) - 1u;
                uint32_t mine = 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t d = sgn ? dropped2<true>(v[i], pk) : dropped2<false>(v[i], pk);
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const unsigned long long m = __ballot(in && !((d >> (16 * e)) & 1u));
                        const uint32_t half = lane < 32 ? (uint32_t)m : (uint32_t)(m >> 32);
                        if ((lane & 31) == 2 * i + e) mine = half;
                    }
                }
                if ((pj.mask_mode & kMaskUnion) && mine) mine = all_tokens;
                if ((lane & 31) < 8 && c < d_in) pj.chan_bits[c + (lane & 31)] = mine;
            }
        }
    }

    f32x4 acc[NB][NF];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[i][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint32_t want = is_t ? 0xffffffffu : 0u;
#define RS_STREAM(MODE) stream_rows<DT, NB, NF, MODE>(mat, aoff, x, xoff, sx, kp, want, lane, d_in, lo + w, hi, nw, va, acc)
    switch (jb.mask_mode) {
    case kMaskNone: RS_STREAM(kMaskNone); break;
    case kMaskOwn: RS_STREAM(kMaskOwn); break;
    case kMaskUnion: RS_STREAM(kMaskUnion); break;
    case kMaskOwn | kMaskSigned: RS_STREAM(kMaskOwn | kMaskSigned); break;
    default: RS_STREAM(kMaskUnion | kMaskSigned); break;
    }
#undef RS_STREAM
    const bool lowrank = !is_t && jb.t_blocks > 0, hand_off = lowrank && ga.phases == 3;

    // the waves meet in LDS; sum_up adds up item (tile, lane)
    auto meet = [&]() {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int f = 0; f < NF; ++f) *reinterpret_cast<f32x4 *>(sx + (i * NF + f) * 1024 + lane * 16) = acc[i][f];
        __syncthreads();
    };
    auto sum_up = [&](int item) {
        f32x4 s = *reinterpret_cast<const f32x4 *>(smem + item * 16);
        for (int ww = 1; ww < nw; ++ww) s += *reinterpret_cast<const f32x4 *>(smem + (size_t)ww * kWaveLds + item * 16);
        return s;
    };

    if (is_t) {
        // ---- t: one wave sums the waves up; with several slices it adds to t_acc, and the last slice to arrive takes the
        //      sums out again (which leaves zeros); they are split and published
        meet();
        if (w == 0) {
            f32x4 s[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) s[f] = sum_up(f * 64 + lane);
            bool mine = true;
            if (ga.t_slices > 1) {
                float *ta = jb.t_acc + (size_t)unit * NF * 256 + lane;
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        __hip_atomic_fetch_add(ta + f * 256 + j * 64, s[f][j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                wait_own_writes();
                int *ctr = jb.t_flags + t_flag_pitch(jb.rank) + unit;
                int arrived = 0;
                if (lane == 0) arrived = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                mine = uniform(arrived) == ga.t_slices - 1;
                if (mine) {
                    if (lane == 0) __hip_atomic_store(ctr, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int f = 0; f < NF; ++f)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            s[f][j] = __hip_atomic_exchange(ta + f * 256 + j * 64, 0.f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if (mine) {
                const int row = unit * 16 + 4 * (lane >> 4);
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    // rank indices row..row+3 of a token, in operand layout; entries past the rank are zero
                    uint32_t hi[2] = {0, 0}, lw[2] = {0, 0};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float v = row < jb.rank ? s[f][e] : 0.f;
                        const uint16_t hb = narrow<DT>(v);
                        hi[e >> 1] |= (uint32_t)hb << (16 * (e & 1));
                        lw[e >> 1] |= (uint32_t)narrow<DT>((v - widen16<DT>(hb)) * LoScale<DT>::value) << (16 * (e & 1));
                    }
                    const int r = row % kMfmaK;
                    unsigned char *p = jb.t + (size_t)(row / kMfmaK * NF + f) * 2048 + (size_t)((r / 8) * 16 + (lane & 15)) * 16 + (r % 8) * 2;
                    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), (unsigned long long)hi[0] | ((unsigned long long)hi[1] << 32),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p + 1024), (unsigned long long)lw[0] | ((unsigned long long)lw[1] << 32),
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (ga.phases == 3) {
                    wait_own_writes();                           // performed: now the block counts as ready
                    if (lane == 0 && !ga.skip_stage1)
                        __hip_atomic_store(jb.t_flags + unit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        return;
    }

    // ---- U_r t: the rank's steps of 32, one per wave in turn; the rows of U_r are requested before t is waited for
    if (lowrank) {
        f32x4 ah[NB][NF], al[NB][NF];                          // the products with t's hi and lo halves
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int f = 0; f < NF; ++f) ah[i][f] = al[i][f] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int usteps = (jb.rank + kMfmaK - 1) / kMfmaK;
        const size_t ublock = (size_t)usteps * 1024;
        const unsigned char *um = reinterpret_cast<const unsigned char *>(jb.U) + (size_t)block0 * ublock + lane * 16;
        constexpr int US = NB * NF == 1 ? 4 : 2;
        u32x4 ua[US][NB];
        auto request_u = [&](int s0) {
#pragma unroll
            for (int u = 0; u < US; ++u) {
                const int s = min(s0 + u * nw, usteps - 1);
#pragma unroll
                for (int i = 0; i < NB; ++i)
                    ua[u][i] = ld16(um + min(i, n_blocks - 1 - block0) * ublock + (size_t)s * 1024);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        request_u(w);
        if (hand_off) {
            // one wave looks at the flags (every block of t has one of its own: no read-modify-write, so nothing
            // queues up on them), the others wait for it at the barrier
            if (w == 0) {
                const long long t0 = wall_clock64();
                bool ok = false;
                for (int polls = 0; polls < ga.wait_polls && !ok; ++polls) {
                    ok = true;
                    for (int i = lane; i < jb.t_blocks; i += 64)
                        ok = ok && __hip_atomic_load(jb.t_flags + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
                    ok = __all(ok);
                    if (!ok) {
                        __builtin_amdgcn_s_sleep(16);
                        if (wall_clock64() - t0 > kWaitLimitTicks) break;
                    }
                }
                if (!ok && lane == 0) __hip_atomic_store(jb.sync + kSyncError, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            __atomic_signal_fence(__ATOMIC_ACQUIRE);           // no load of t moves up here
        }
        for (int s0 = w; s0 < usteps; s0 += nw * US) {
            u32x4 th[US][NF], tl[US][NF];
#pragma unroll
            for (int u = 0; u < US; ++u) {
                const int s = min(s0 + u * nw, usteps - 1);
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    const unsigned char *p = jb.t + (size_t)(s * NF + f) * 2048 + lane * 16;
                    th[u][f] = *reinterpret_cast<const u32x4 *>(p);
                    tl[u][f] = *reinterpret_cast<const u32x4 *>(p + 1024);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < US; ++u) {
                if (s0 + u * nw < usteps) {
#pragma unroll
                    for (int i = 0; i < NB; ++i)
#pragma unroll
                        for (int f = 0; f < NF; ++f) {
                            ah[i][f] = mfma16<DT>(ua[u][i], th[u][f], ah[i][f]);
                            al[i][f] = mfma16<DT>(ua[u][i], tl[u][f], al[i][f]);
                        }
                }
            }
            if (s0 + nw * US < usteps) request_u(s0 + nw * US);
        }
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][f][j] += ah[i][f][j] + al[i][f][j] * (1.0f / LoScale<DT>::value);
    }

    meet();
    // every wave of this workgroup has read t: count the unit, over kTReadSubs counters first, so that the units, which end
    // together, do not queue up on one address (the answer is looked at after the stores)
    const bool counted = hand_off && tid == 0;
    const int sub = unit % kTReadSubs;
    int *const t_read = jb.t_flags + 2 * t_flag_pitch(jb.rank);
    int arrived = -1;
    if (counted) arrived = __hip_atomic_fetch_add(t_read + sub * 32, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int item = tid; item < kTiles * 64; item += nthr) {
        const int l = item & 63, tile = item >> 6, i = tile / NF, f = tile % NF;
        const f32x4 s = sum_up(item);
        const int tok = f * 16 + (l & 15);
        const int row = (block0 + i) * 16 + 4 * (l >> 4);       // four consecutive rows (d_out is a multiple of 8)
        if (tok < batch && row < jb.d_out) {
            float o[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = jb.bias ? s[j] + jb.bias[row + j] : s[j];
            const size_t oi = (size_t)tok * jb.d_out + row;
            if (jb.out_dtype == F32) {
                *reinterpret_cast<float4 *>((float *)jb.Y + oi) = float4{o[0], o[1], o[2], o[3]};
            } else {
                uint2 pk;
                pk.x = (uint32_t)narrow<DT>(o[0]) | ((uint32_t)narrow<DT>(o[1]) << 16);
                pk.y = (uint32_t)narrow<DT>(o[2]) | ((uint32_t)narrow<DT>(o[3]) << 16);
                *reinterpret_cast<uint2 *>((uint16_t *)jb.Y + oi) = pk;
            }
        }
    }
    if (counted && arrived == (jb.w_units - sub + kTReadSubs - 1) / kTReadSubs - 1) {
        // the last of its counter; the last of the counters puts the flags back for the next call
        __hip_atomic_store(t_read + sub * 32, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__hip_atomic_fetch_add(t_read + 32 * kTReadSubs, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == min(jb.w_units, kTReadSubs) - 1) {
            __hip_atomic_store(t_read + 32 * kTReadSubs, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int i = 0; i < jb.t_blocks; ++i) __hip_atomic_store(jb.t_flags + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

}  // namespace

bool mfma_path_supported(const MatrixView &M, int batch) { return batch >= 1 && batch <= 32 && M.W != nullptr; }

size_t mfma_operand_bytes(size_t rows, size_t cols, size_t row_pad)
{
    return (rows + row_pad - 1) / row_pad * (row_pad / 16) * ((cols + kMfmaK - 1) / kMfmaK) * 1024;
}

// One thread per 16 bytes of the result.
__global__ void k_pack_operand(const uint16_t *src, size_t rows, size_t cols, size_t steps, uint16_t *dst, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const size_t l = i % 64, tile = i / 64, row = tile / steps * 16 + l % 16, col = tile % steps * kMfmaK + l / 16 * 8;
        u32x4 v = u32x4{0, 0, 0, 0};
        if (row < rows && col < cols) v = *reinterpret_cast<const u32x4 *>(src + row * cols + col);
        *reinterpret_cast<u32x4 *>(dst + i * 8) = v;
    }
}

hipError_t launch_pack_operand(const uint16_t *src, size_t rows, size_t cols, size_t row_pad, uint16_t *dst, hipStream_t stream)
{
    const size_t n = mfma_operand_bytes(rows, cols, row_pad) / 16, steps = (cols + kMfmaK - 1) / kMfmaK;
    hipLaunchKernelGGL(k_pack_operand, dim3((unsigned)std::min<size_t>((n + 255) / 256, 16384)), dim3(256), 0, stream, src, rows, cols, steps, dst, n);
    return hipGetLastError();
}

size_t mfma_t_bytes(int rank) { return (size_t)((rank + kMfmaK - 1) / kMfmaK) * 2 * 2048; }

// 64 x 64 tiles through LDS, 16 bytes per access on both sides.
__global__ __launch_bounds__(256) void k_transpose16(const uint16_t *src, size_t rows, size_t cols, uint16_t *dst)
{
    __shared__ uint16_t tile[64][66];
    const size_t c0 = (size_t)blockIdx.x * 64, r0 = (size_t)blockIdx.y * 64;
    for (int i = threadIdx.x; i < 512; i += 256) {
        const size_t r = r0 + i / 8, c = c0 + i % 8 * 8;
        if (r < rows && c < cols) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(src + r * cols + c);
#pragma unroll
            for (int e = 0; e < 8; ++e) tile[i / 8][i % 8 * 8 + e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 512; i += 256) {
        const size_t c = c0 + i / 8, r = r0 + i % 8 * 8;
        if (c < cols && r < rows) {
            u32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (uint32_t)tile[i % 8 * 8 + 2 * e][i / 8] | ((uint32_t)tile[i % 8 * 8 + 2 * e + 1][i / 8] << 16);
            *reinterpret_cast<u32x4 *>(dst + c * rows + r) = v;
        }
    }
}

hipError_t launch_transpose16(const uint16_t *src, size_t rows, size_t cols, uint16_t *dst, hipStream_t stream)
{
    if (rows == 0 || cols == 0) return hipSuccess;
    hipLaunchKernelGGL(k_transpose16, dim3((unsigned)((cols + 63) / 64), (unsigned)((rows + 63) / 64)), dim3(256), 0, stream, src, rows, cols, dst);
    return hipGetLastError();
}

hipError_t launch_mfma(const LayerView *L, const MatrixView *M, int n, const void *X, int batch, void *const *Y, uint32_t *const *chan_bits, int cus,
                       int phases, bool dense, int rows_per_wg_hint, int wait_polls, int skip_stage1, hipStream_t stream)
{
    if (n < 1 || n > kMaxGroupLayers || batch < 1 || batch > 32 || phases < 1 || phases > 3) return hipErrorInvalidValue;
    const int nf = batch > 16 ? 2 : 1;
    MfmaArgs a{};
    a.n = n; a.X = (const uint16_t *)X; a.batch = batch; a.d_in = L[0].d_in; a.phases = phases;
    a.wait_polls = wait_polls > 0 ? wait_polls : kWaitLimitPolls;
    a.skip_stage1 = skip_stage1;
    // Units of one block for up to 16 tokens, of two for more (a unit reads all tokens, from L2, beside its rows: at 32
    // tokens and one block twice the bytes of the rows; measured at 8192 x 8192, 32 tokens: dense 33.7 us with one block,
    // 27.0 with two; at 8 tokens 23.2 and 22.9, at 4096 -> 14336 with 16 tokens 70.9 and 78.1) -- unless that leaves
    // compute units without a unit.  Four waves a unit: with eight the same bytes are in flight in half the workgroups
    // (8192 x 8192, 8 tokens: 24.7 against 25.8 us).
    int nb = 1, nw = 4;
    if (nf == 2) {
        int blocks = 0;
        for (int i = 0; i < n; ++i) blocks += (L[i].d_out + 15) / 16;
        if (blocks >= 2 * cus || rows_per_wg_hint > 0) nb = 2;
    }
    int w_total = 0, t_blocks = 0;
    for (int i = 0; i < n; ++i) {
        MfmaJob &jb = a.job[i];
        const LayerView &v = L[i];
        const MatrixView &m = M[i];
        if (v.d_in != a.d_in || v.dtype != L[0].dtype || !mfma_path_supported(m, batch) || !Y[i]) return hipErrorInvalidValue;
        jb.W = m.W; jb.SVt = m.SVt; jb.U = m.U; jb.t = (unsigned char *)m.t; jb.Y = Y[i]; jb.bias = v.bias;
        jb.t_acc = m.t_acc; jb.t_flags = m.t_flags;
        jb.chan_bits = dense ? nullptr : chan_bits[i];
        jb.sync = v.sync; jb.d_out = v.d_out; jb.rank = dense ? 0 : v.rank; jb.out_dtype = v.out_dtype;
        jb.mask_mode = dense ? kMaskNone : (v.batch_mask_mode == 1 ? kMaskUnion : kMaskOwn) | (v.keep_signed ? kMaskSigned : 0);
        jb.kp = KeepPattern{(uint32_t)(uint16_t)m.keep_min * 0x10001u, (v.dtype == F16 ? 0x7c00u : 0x7f80u) * 0x10001u};
        if (jb.rank > 0 && (!m.t || !m.t_acc || !v.sync || !m.t_flags || !m.SVt || !m.U)) return hipErrorInvalidValue;
        jb.t_blocks = (jb.rank + 31) / 32 * 2;
        jb.w_units = ((v.d_out + 15) / 16 + nb - 1) / nb;
        w_total += jb.w_units;
        t_blocks += jb.t_blocks;
        a.w_end[i] = w_total;
    }
    const int batch_k = kMfmaK * (nb == 1 ? 4 : 2), n_batches = (a.d_in + batch_k - 1) / batch_k;
    // K slices of t: enough workgroups for the chip, a batch of loads for every wave, and at most four, whose sums meet in
    // atomics (8192 x 8192, rank 1024, 8 tokens: 43.5 us with one slice, 39.0 with two, 34.5 with four; 4096 x 4096, rank
    // 256: 16.1 with one, 14.6 with four, 15.4 with sixteen)
    a.t_slices = t_blocks > 0 ? std::max(1, std::min({4, cus / t_blocks, n_batches / nw})) : 1;
    int t_total = 0;
    for (int i = 0; i < kMaxGroupLayers; ++i) {
        if (i < n) t_total += a.job[i].t_blocks * a.t_slices;
        else a.w_end[i] = w_total;
        a.t_end[i] = t_total;
    }
    if (phases == 1 && t_total == 0) return hipSuccess;
    const size_t lds = (size_t)nw * std::max(nf * 16 * (batch_k * 2 + 16), nb * nf * 1024);
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    dim3 grid((phases & 1 ? t_total : 0) + (phases & 2 ? w_total : 0)), block(64 * nw);
#define RS_M(DT, NBV, NFV) hipLaunchKernelGGL((k_mfma_rows<DT, NBV, NFV>), grid, block, lds, stream, a)
#define RS_MD(DT)                                                                               \
    do {                                                                                        \
        if (nf == 1) RS_M(DT, 1, 1);                                                            \
        else if (nb == 1) RS_M(DT, 1, 2);                                                       \
        else RS_M(DT, 2, 2);                                                                    \
    } while (0)
    if (L[0].dtype == F16) RS_MD(F16); else RS_MD(BF16);
#undef RS_MD
#undef RS_M
    return hipGetLastError();
}

}  // namespace rsparse
