// Matrix-core kernel over column-major W (layers without the operand-layout copy): yc += X' W^T, X' the kept part of the
// tokens (all of them for the dense product), up to 32 tokens in one pass over W.
//
// The vector kernels hold at most 8 tokens and spend an FMA per weight and token; from a few tokens on the union of kept
// channels is nearly all of them anyway, so W is streamed whole, once.  v_mfma_f32_16x16x32 wants 8 consecutive channels
// of one output per lane, column-major W has 8 outputs of one channel in 16 bytes: a lane loads the same 8 outputs of 8
// channels (16 lanes cover 256 bytes of a channel) and turns the 8 x 8 values with one byte permute per two of them.  A
// wave's tile is 128 outputs x 32 channels a step, 8 MFMAs per 16 tokens.  A workgroup of four waves takes a K slice of a
// unit of 128 outputs; slices meet in fp32 atomics on yc.  The workgroups of t stand at the front of the grid; U_r t, the
// sum and the rounding are the next launch's (k_mfma_rows without a W part).  Bound by HBM.
// Measured (gate, up and down at 4096 / 11008, rank 512, f16, us, vector kernels in tiles of 8 tokens -> this): 125 -> 72 at
// 5 tokens, 234 -> 75 at 16, 389 -> 95 at 32; of the 75, 59 are the two launches of this kernel (270 MB at 7 TB/s: 39).
#include "device_mfma.h"

#include <algorithm>

namespace rsparse {
namespace {

constexpr int kColWaves = 4, kColOuts = 128, kChain = 8;

struct ColsJob {
    MfmaJob t;                   // its t part, mask, yc, d_out
    const uint16_t *M;           // [d_in ...][d_out]
    int units, splits;
};
struct ColsArgs {
    ColsJob job[kMaxGroupLayers];
    int t_end[kMaxGroupLayers], w_end[kMaxGroupLayers];
    const uint16_t *X;
    int batch, d_in, t_slices;
};

template <int NF>
struct ColsStep {
    u32x4 c[8], x[NF];           // channel 8 g + c of the step: 8 outputs; the lane's 8 channels of token lane % 16
};

template <int DT, int NF>
__global__ __launch_bounds__(64 * kColWaves, 2) void k_mfma_cols(const ColsArgs ga)
{
    // t's staging, or the waves' sums of half the unit's outputs [wave][64][16 * NF]
    constexpr int kLds = kColWaves * (kColOuts / 2) * 16 * NF * 4, kLdsT = kColWaves * t_unit_lds<NF>;
    __shared__ __align__(16) unsigned char smem[kLds > kLdsT ? kLds : kLdsT];
    const int t_wgs = ga.t_end[kMaxGroupLayers - 1];
    const bool is_t = (int)blockIdx.x < t_wgs;
    const int first = is_t ? (int)blockIdx.x : (int)blockIdx.x - t_wgs;
    int job = 0, begin = 0;
#pragma unroll
    for (int j = 0; j < kMaxGroupLayers - 1; ++j) {
        const int e = is_t ? ga.t_end[j] : ga.w_end[j];
        if (first >= e) { job = j + 1; begin = e; }
    }
    const ColsJob &cj = ga.job[job];
    const int d_in = ga.d_in, batch = ga.batch;
    if (is_t) {
        t_unit<DT, NF, false>(cj.t, ga.X, batch, d_in, (first - begin) / ga.t_slices, (first - begin) % ga.t_slices, ga.t_slices, false, 0, smem);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, w = uniform(tid >> 6), i16 = lane & 15, g4 = lane >> 4;
    const int unit = (first - begin) / cj.splits, split = (first - begin) % cj.splits;
    const int d_out = cj.t.d_out, col0 = unit * kColOuts, mode = cj.t.mask_mode;
    const KeepPattern kp = cj.t.kp;
    // (outputs past the matrix and tokens past the batch repeat the last ones; their results are not used)
    const uint16_t *const M = cj.M + min(col0 + i16 * 8, d_out - 8);
    const uint16_t *xrow[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) xrow[f] = ga.X + (size_t)min(f * 16 + i16, batch - 1) * d_in;

    int lo, hi, w_lo, w_hi;
    balanced_share((d_in + kMfmaK - 1) / kMfmaK, cj.splits, split, lo, hi);
    balanced_share(hi - lo, kColWaves, w, w_lo, w_hi);
    w_lo += lo;
    w_hi += lo;

    auto load = [&](int s, ColsStep<NF> &v) {
        const int ch = s * kMfmaK + g4 * 8, chx = min(ch, d_in - 8);    // (the last step may lie partly past d_in)
#pragma unroll
        for (int f = 0; f < NF; ++f) v.x[f] = *reinterpret_cast<const u32x4 *>(xrow[f] + chx);
        const uint16_t *p = M + (size_t)chx * d_out;
#pragma unroll
        for (int c = 0; c < 8; ++c) v.c[c] = ldg16<true>(p + (size_t)c * d_out);
        __builtin_amdgcn_sched_barrier(0);
    };
    // Long chains of sums inside the matrix cores lose bits: every kChain steps they go over to the vector ALU.  Two token
    // tiles have no registers for that; the host then gives no wave more than 2 * kChain steps.
    constexpr bool kFlush = NF == 1;
    f32x4 acc[kFlush ? 8 : 1][NF], sum[8][NF];
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[kFlush ? e : 0][f] = sum[e][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto use = [&](ColsStep<NF> &v, int s) {
        switch (mode) {
        case kMaskNone: break;
        case kMaskOwn: mask_step<NF, kMaskOwn>(v.x, kp, 0u); break;
        case kMaskUnion: mask_step<NF, kMaskUnion>(v.x, kp, 0u); break;
        case kMaskOwn | kMaskSigned: mask_step<NF, kMaskOwn | kMaskSigned>(v.x, kp, 0u); break;
        default: mask_step<NF, kMaskUnion | kMaskSigned>(v.x, kp, 0u); break;
        }
        if (s * kMfmaK + g4 * 8 >= d_in) {
#pragma unroll
            for (int f = 0; f < NF; ++f) v.x[f] = u32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            u32x4 a;
#pragma unroll
            for (int p = 0; p < 4; ++p)
                a[p] = __builtin_amdgcn_perm(v.c[2 * p + 1][e >> 1], v.c[2 * p][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
            for (int f = 0; f < NF; ++f) sum[e][f] = mfma16<DT>(a, v.x[f], sum[e][f]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto flush = [&]() {
        if constexpr (kFlush) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int f = 0; f < NF; ++f) { acc[e][f] += sum[e][f]; sum[e][f] = f32x4{0.f, 0.f, 0.f, 0.f}; }
        }
    };
    if (w_lo < w_hi) {
        ColsStep<NF> va, vb;
        load(w_lo, va);
        for (int s = w_lo; s < w_hi; s += 2) {
            load(min(s + 1, w_hi - 1), vb);
            use(va, s);
            if (s + 1 >= w_hi) break;
            load(min(s + 2, w_hi - 1), va);
            use(vb, s + 1);
            if (((s - w_lo) & (kChain - 1)) == kChain - 2) flush();
        }
    }
    flush();

    // ---- the waves meet in LDS, half the outputs at a time: [wave][token tile][64 outputs][16 tokens]
    float *red = reinterpret_cast<float *>(smem);
    constexpr int kHalf = 64 * 16 * NF;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        __syncthreads();
        if ((g4 >> 1) == h) {                                   // rows 4 g4 + r of tile e: output 8 (4 g4 + r) + e
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int r = 0; r < 4; ++r) red[w * kHalf + (f * 64 + ((g4 & 1) * 4 + r) * 8 + e) * 16 + i16] = (kFlush ? acc[kFlush ? e : 0] : sum[e])[f][r];
        }
        __syncthreads();
        for (int i = tid; i < kHalf; i += 64 * kColWaves) {
            const int f = i / 1024, o = col0 + h * 64 + i % 1024 / 16;
            float s = red[i];
#pragma unroll
            for (int ww = 1; ww < kColWaves; ++ww) s += red[ww * kHalf + i];
            if (o < d_out && f * 16 + (i & 15) < batch)
                __hip_atomic_fetch_add(cj.t.yc + ((size_t)f * cj.t.yc_rows + o) * 16 + (i & 15), s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

}  // namespace

hipError_t launch_mfma_cols(const LayerView *L, const MatrixView *M, int n, const void *X, int batch, bool dense, int cus, hipStream_t stream)
{
    if (n < 1 || n > kMaxGroupLayers || batch < 1 || batch > 32) return hipErrorInvalidValue;
    ColsArgs a{};
    a.X = (const uint16_t *)X; a.batch = batch; a.d_in = L[0].d_in;
    int t_blocks = 0, units = 0;
    for (int i = 0; i < n; ++i) {
        if (!L[i].M || !M[i].yc || L[i].d_in != a.d_in || L[i].dtype != L[0].dtype) return hipErrorInvalidValue;
        ColsJob &c = a.job[i];
        MfmaJob &j = c.t;
        c.M = L[i].M;
        c.units = (L[i].d_out + kColOuts - 1) / kColOuts;
        units += c.units;
        j.yc = M[i].yc; j.yc_rows = M[i].yc_rows; j.d_out = L[i].d_out; j.rank = dense ? 0 : L[i].rank;
        j.mask_mode = dense ? kMaskNone : (L[i].batch_mask_mode == 1 ? kMaskUnion : kMaskOwn) | (L[i].keep_signed ? kMaskSigned : 0);
        j.kp = KeepPattern{(uint32_t)(uint16_t)M[i].keep_min * 0x10001u, (L[i].dtype == F16 ? 0x7c00u : 0x7f80u) * 0x10001u};
        j.SVt = M[i].SVt; j.t = (unsigned char *)M[i].t; j.t_acc = M[i].t_acc; j.t_flags = M[i].t_flags;
        if (j.rank > 0 && (!j.SVt || !j.t || !j.t_acc || !j.t_flags)) return hipErrorInvalidValue;
        j.t_blocks = (j.rank + 31) / 32 * 2;
        t_blocks += j.t_blocks;
    }
    a.t_slices = mfma_t_slices(t_blocks, a.d_in, kColWaves, cus);
    // K slices: about one workgroup per compute unit over the launch (gate, up and down at 4096 / 11008, 12 tokens: 78 us; 88
    // at twice as many, whose sums cost more), and no wave with a longer chain of sums than it may have
    const int steps = (a.d_in + kMfmaK - 1) / kMfmaK, min_splits = batch > 16 ? (steps + 2 * kChain * kColWaves - 1) / (2 * kChain * kColWaves) : 1;
    int t_total = 0, w_total = 0;
    for (int i = 0; i < kMaxGroupLayers; ++i) {
        if (i < n) {
            t_total += a.job[i].t.t_blocks * a.t_slices;
            a.job[i].splits = std::max({1, min_splits, std::min((cus + units / 2) / units, steps / kColWaves)});
            w_total += a.job[i].units * a.job[i].splits;
        }
        a.t_end[i] = t_total;
        a.w_end[i] = w_total;
    }
    dim3 grid(t_total + w_total), block(64 * kColWaves);
    if (L[0].dtype == F16) {
        if (batch <= 16) hipLaunchKernelGGL((k_mfma_cols<F16, 1>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((k_mfma_cols<F16, 2>), grid, block, 0, stream, a);
    } else {
        if (batch <= 16) hipLaunchKernelGGL((k_mfma_cols<BF16, 1>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((k_mfma_cols<BF16, 2>), grid, block, 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace rsparse
