// Device code shared by the matrix-core kernel files: the MFMA itself, operand types, and the sparsification function on
// packed 16-bit patterns.
#pragma once
#include "kernels.h"
#include "device_common.h"
#include "device_stage1.h"

namespace rsparse {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

constexpr int kMfmaK = 32;        // contraction depth of one MFMA

template <int DT>
__device__ __forceinline__ f32x4 mfma16(const u32x4 a, const u32x4 b, const f32x4 c)
{
    if (DT == BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// acc += A B for 8 consecutive k per lane (a: 16-bit, b: fp32), each product and sum in fp32: what a 16-bit operand cannot hold of b.
template <int DT>
__device__ __forceinline__ f32x4 mfma_f32(const u32x4 a, const f32x4 (&b)[2], f32x4 acc)
{
    float f[8];
    unpack8<DT>(a, f);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(f[e], b[e >> 2][e & 3], acc, 0, 0, 0);
    return acc;
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

// MFMA steps of one batch of loads, for units of NB blocks and NF token tiles.  Measured on plain streams of this shape (512 workgroups of
// 8 waves, 134 MB): two batches of 4 KiB per wave in flight 6.3 TB/s, of 8 KiB 5.6, of 16 KiB 4.5 -- more requests than
// the memory system takes only push each other out.
template <int NB, int NF> struct StepsOf { static constexpr int value = NB * NF == 1 ? 4 : 2; };

// Bytes of the 16-bit parts of t in its buffer; t in fp32 follows and takes as many.
__host__ __device__ inline size_t t32_offset(int rank) { return (size_t)((rank + kMfmaK - 1) / kMfmaK) * 2 * 2 * 1024; }

struct MfmaJob {
    const uint16_t *W, *SVt, *U; // operand layout (MatrixView)
    unsigned char *t;            // t in two 16-bit parts: [step of 32 rank indices][token tile][part][64 lanes][16 bytes], and
                                 // from t32_offset(rank) on as it is: [step of 32 rank indices][token tile][64 lanes][8] floats
    float *t_acc;                // [block of 16 rank indices][token tile][4][64] fp32 sums of t's K slices, zero between calls
    int *t_flags;                // a flag per block of t, zero between calls; then an arrival counter per block
    void *Y;
    const float *bias;
    float *yc;                   // sums of the W part from an earlier launch, [token tile][yc_rows][16], put back to zero (W == nullptr)
    int yc_rows;
    uint32_t *chan_bits;         // [d_in] bit b = token b keeps the channel (read-back), or nullptr
    int *sync;
    int d_out, rank;
    int out_dtype, mask_mode;
    KeepPattern kp;
    int t_blocks, w_units;       // blocks of S_r V_r^T (0: no low-rank part), units of W
    __device__ float *t32() const { return reinterpret_cast<float *>(t + t32_offset(rank)); }
};
// One batch of a wave: S steps of NB weight tiles (1 KiB each) and the same 32 * S channels of all tokens, 4 * S lanes to
// a token.
template <int NB, int NF>
struct Batch {
    static constexpr int S = StepsOf<NB, NF>::value, K = kMfmaK * S, kLanes = 4 * S, kX = NF * S;
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

// A unit of t: block `unit` of 16 rank indices over K slice `slice` of t_slices, by all waves of a workgroup (nw *
// t_unit_lds<NF> bytes of LDS).  One wave sums the waves up; with several slices it adds to t_acc, and the last slice to
// arrive takes the sums out again (which leaves zeros).  They are stored as they are (PARTS = false), or in two 16-bit parts
// -- in fp16, whose range t can leave, as they are besides.  flags: the block's flag is set when the stores have been
// performed, for readers in the same launch.
template <int NF>
constexpr int t_unit_lds = NF * 16 * Batch<1, NF>::kPitch;

template <int DT, int NF, bool PARTS>
__device__ __forceinline__ void t_unit(const MfmaJob &jb, const uint16_t *X, int batch, int d_in, int unit, int slice, int t_slices, bool flags,
                                       int skip_flag, unsigned char *smem)
{
    using B = Batch<1, NF>;
    const int tid = threadIdx.x, lane = tid & 63, w = uniform(tid >> 6), nw = uniform((int)blockDim.x >> 6);
    const int steps = (d_in + kMfmaK - 1) / kMfmaK, n_batches = (steps + B::S - 1) / B::S;
    const unsigned char *x = reinterpret_cast<const unsigned char *>(X);
    const unsigned char *mat = reinterpret_cast<const unsigned char *>(jb.SVt) + (size_t)unit * steps * 1024;
    const KeepPattern kp = jb.kp;
    uint32_t xoff[B::kX];
#pragma unroll
    for (int j = 0; j < B::kX; ++j) xoff[j] = (uint32_t)min(j * (64 / B::kLanes) + lane / B::kLanes, batch - 1) * (uint32_t)d_in * 2u;
    unsigned char *sx = smem + (size_t)w * t_unit_lds<NF>;
    const int lo = (int)((unsigned)(n_batches * slice) / (unsigned)t_slices), hi = (int)((unsigned)(n_batches * (slice + 1)) / (unsigned)t_slices);
    const size_t aoff[1] = {0};
    f32x4 acc[1][NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[0][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    Batch<1, NF> va;
    load_batch<1, NF>(mat, aoff, x, xoff, lane, d_in, steps, lo + w, va);
#define RS_STREAM(MODE) stream_rows<DT, 1, NF, MODE>(mat, aoff, x, xoff, sx, kp, 0xffffffffu, lane, d_in, lo + w, hi, nw, va, acc)
    switch (jb.mask_mode) {
    case kMaskOwn: RS_STREAM(kMaskOwn); break;
    case kMaskUnion: RS_STREAM(kMaskUnion); break;
    case kMaskOwn | kMaskSigned: RS_STREAM(kMaskOwn | kMaskSigned); break;
    default: RS_STREAM(kMaskUnion | kMaskSigned); break;
    }
#undef RS_STREAM
#pragma unroll
    for (int f = 0; f < NF; ++f) *reinterpret_cast<f32x4 *>(sx + f * 1024 + lane * 16) = acc[0][f];
    __syncthreads();
    auto sum_up = [&](int item) {
        f32x4 s = *reinterpret_cast<const f32x4 *>(smem + item * 16);
        for (int ww = 1; ww < nw; ++ww) s += *reinterpret_cast<const f32x4 *>(smem + (size_t)ww * t_unit_lds<NF> + item * 16);
        return s;
    };
    if (w == 0) {
        f32x4 s[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) s[f] = sum_up(f * 64 + lane);
        bool mine = true;
        if (t_slices > 1) {
            float *ta = jb.t_acc + (size_t)unit * NF * 256 + lane;
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    __hip_atomic_fetch_add(ta + f * 256 + j * 64, s[f][j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wait_own_writes();
            int *ctr = jb.t_flags + t_arrival(jb.rank, unit);
            int arrived = 0;
            if (lane == 0) arrived = __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            mine = uniform(arrived) == t_slices - 1;
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
                const int r = row % kMfmaK, at = r / 8 * 16 + (lane & 15);
                const f32x4 v4 = row < jb.rank ? s[f] : f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (!PARTS || DT == F16) {
                    unsigned long long *p = reinterpret_cast<unsigned long long *>(jb.t32() + ((size_t)(row / kMfmaK * NF + f) * 64 + at) * 8 + r % 8);
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        __hip_atomic_store(p + h, (unsigned long long)as_u(v4[2 * h]) | ((unsigned long long)as_u(v4[2 * h + 1]) << 32), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                }
                if constexpr (PARTS) {
                    constexpr uint32_t kInf = DT == F16 ? 0x7c00u : 0x7f80u;
                    unsigned long long part[2] = {};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float v = v4[e];
                        const uint16_t hi = narrow<DT>(v);
                        // the second part rounds what the first left over (exact); nothing is left over of an infinity
                        const float rest = (hi & kInf) == kInf ? 0.f : (v - widen16<DT>(hi)) * LoScale<DT>::value;
                        part[0] |= (unsigned long long)hi << (16 * e);
                        part[1] |= (unsigned long long)narrow<DT>(rest) << (16 * e);
                    }
                    unsigned char *p = jb.t + (size_t)(row / kMfmaK * NF + f) * 2048 + (size_t)at * 16 + (r % 8) * 2;
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        __hip_atomic_store(reinterpret_cast<unsigned long long *>(p + h * 1024), part[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if (flags) {
                wait_own_writes();                           // performed: now the block counts as ready
                if (lane == 0 && !skip_flag)
                    __hip_atomic_store(jb.t_flags + unit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

}  // namespace
}  // namespace rsparse
