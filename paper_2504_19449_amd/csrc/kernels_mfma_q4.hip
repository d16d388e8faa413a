// Matrix-core kernel for 4-bit weights (R-Sparse, Sec. 4.4) from 3 tokens on: yc += X' (q - z) s over the
// channel-major codes (layout: LayerView::Mq), X' the kept part of the tokens (all of them for the dense product).
//
// The union of kept channels is most of them (nearly all from 4 tokens on), so every channel is streamed, once for 16
// tokens -- the vector kernel streams the codes once per 4 tokens and spends an FMA per code and token (16 tokens, 4096 <-> 11008:
// 240 us per layer).  v_mfma_f32_16x16x32 wants 8 consecutive channels of one output per lane, the layout has 16 outputs
// of one channel: a lane loads the same 16 outputs of 8 channels (8 loads of 8 bytes; 16 lanes cover 128 bytes of a
// channel) and turns the 8 x 16 codes in registers, where converting and turning are the same instructions: per pair of
// channels one byte permute (fp16; 1024 + code by OR, then one packed operation) or two conversions and one permute
// (bf16: a code's fp32 pattern ends in 16 zeros, so its upper half is exact).  A wave's tile is 256 outputs x 32 channels
// a step: 16 MFMAs, and one more against ones, which gives sum_c x_c in the layout of the results.  Per quantisation group
// (or the part of it that a wave has) the sums are folded as s (sum_c x_c q_c - z sum_c x_c) in fp32, as in the vector
// kernel; scales and zero points are requested a group ahead, 12 bytes per lane, and spread through the wave's LDS.
// The workgroups of t stand at the front of the grid; U_r t, the sum and the rounding are the next launch's
// (k_mfma_rows without a W part).
// At full streams it would be bound by the vector ALU (about 2.5 instructions per code in bf16) and HBM in equal parts; at
// decode sizes a wave has 2 to 16 steps and the launch's balance over the compute units counts (launch_mfma_q4).  Gate, up and down at
// 4096 / 11008, rank 512, bf16, 52 us at sixteen tokens and 77 at 32.  Tried and slower, two such blocks at sixteen tokens, 119.4 with the launch
// shape of then: eight waves that share the steps 146, two of them to the eight lane slots of half a unit 142 (128 registers),
// waves side by side on one step 129 to 151 (four times the atomics), three steps in flight 123.
#include "device_mfma.h"

#include <algorithm>

namespace rsparse {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct MfmaQ4Job {
    MfmaJob t;                   // its t part, mask, yc [token tile][yc_rows][16] fp32, added to with atomics
    const uint8_t *Mq, *qz;
    const uint16_t *qs;
    int qtiles, qshift, splits, units;
};
struct MfmaQ4Args {
    MfmaQ4Job job[kMaxGroupLayers];
    int t_end[kMaxGroupLayers];  // workgroups of t of jobs 0..i, at the front of the grid
    int w_end[kMaxGroupLayers];  // workgroups of the codes of jobs 0..i
    const uint16_t *X;
    int d_in, batch, t_slices;
};

// Kept values of one token tile under the union mask of a batch of two tiles.
__device__ __forceinline__ void mask_union_two(u32x4 &mine, u32x4 other, const KeepPattern &kp, bool sgn)
{
    u32x4 b[2] = {mine, other};
    if (sgn) mask_step<2, kMaskUnion | kMaskSigned>(b, kp, 0u);
    else mask_step<2, kMaskUnion>(b, kp, 0u);
    mine = b[0];
}

constexpr int kQ4Waves = 4, kQ4Outs = 256;

// Codes of one step: word h of channel 8 g + c.
struct Q4Step {
    u32x2 c[8];
    u32x4 x;                     // the lane's 8 channels of token lane % 16
};

__device__ __forceinline__ void load_step(const uint8_t *__restrict__ codes, size_t ldq, const uint16_t *__restrict__ xrow, int lane,
                                          int s, Q4Step &v)
{
    const int ch = s * kMfmaK + (lane >> 4) * 8;
    v.x = *reinterpret_cast<const u32x4 *>(xrow + ch);
    const uint8_t *p = codes + (size_t)ch * ldq;
#pragma unroll
    for (int c = 0; c < 8; ++c) v.c[c] = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(p + c * ldq));
    __builtin_amdgcn_sched_barrier(0);
}

// The codes of outputs b (a[0]) and 4 + b (a[1]) of word h for the lane's 8 channels, as 16-bit operands.
template <int DT, int B>
__device__ __forceinline__ void operands(const u32x2 (&c)[8], int h, u32x4 (&a)[2])
{
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t w0 = c[2 * p][h], w1 = c[2 * p + 1][h];
        if (DT == F16) {
            const uint32_t r = __builtin_amdgcn_perm(w1, w0, 0x0c000c00u | (uint32_t)B | ((uint32_t)(4 + B) << 16));   // byte B of both
            const h2 lo = __builtin_bit_cast(h2, (r & 0x000f000fu) | 0x64006400u), hi = __builtin_bit_cast(h2, (r & 0x00f000f0u) | 0x64006400u);
            const h2 k1024 = {(_Float16)-1024.0f, (_Float16)-1024.0f}, k64 = {(_Float16)-64.0f, (_Float16)-64.0f}, k16 = {(_Float16)0.0625f, (_Float16)0.0625f};
            a[0][p] = __builtin_bit_cast(uint32_t, (h2)(lo + k1024));                                  // 1024 + code, exact
            a[1][p] = __builtin_bit_cast(uint32_t, (h2)__builtin_elementwise_fma(hi, k16, k64));       // 1024 + 16 code, exact
        } else {
            const uint32_t l0 = w0 & 0x0f0f0f0fu, l1 = w1 & 0x0f0f0f0fu, h0 = (w0 >> 4) & 0x0f0f0f0fu, h1 = (w1 >> 4) & 0x0f0f0f0fu;
            const uint32_t f0 = as_u((float)((l0 >> (8 * B)) & 0xffu)), f1 = as_u((float)((l1 >> (8 * B)) & 0xffu));
            const uint32_t g0 = as_u((float)((h0 >> (8 * B)) & 0xffu)), g1 = as_u((float)((h1 >> (8 * B)) & 0xffu));
            a[0][p] = __builtin_amdgcn_perm(f1, f0, 0x07060302u);
            a[1][p] = __builtin_amdgcn_perm(g1, g0, 0x07060302u);
        }
    }
}

// NF: token tiles of 16 of the call (for t; a workgroup of the codes takes one tile).
template <int DT, int NF>
__global__ __launch_bounds__(64 * kQ4Waves, 2) void k_mfma_q4(const MfmaQ4Args ga)
{
    // per wave: scales (16-bit) and zero points (bytes) of its 256 outputs; later half the waves' sums [out][token]
    constexpr int kLds = kQ4Waves * kQ4Outs * 16 * 4 / 2, kLdsT = kQ4Waves * t_unit_lds<NF>;
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
    const MfmaQ4Job &a = ga.job[job];
    const int d_in = ga.d_in, batch = ga.batch;
    if (is_t) {
        t_unit<DT, NF, false>(a.t, ga.X, batch, d_in, (first - begin) / ga.t_slices, (first - begin) % ga.t_slices, ga.t_slices, false, 0, smem);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, w = uniform(tid >> 6);
    const int id = first - begin, split = id % a.splits, unit = id / a.splits % a.units, ttile = id / a.splits / a.units, tok0 = ttile * 16;
    const int i16 = lane & 15, g4 = lane >> 4, mode = a.t.mask_mode;
    const KeepPattern kp = a.t.kp;
    const int tile = unit >> 2, lb = (unit & 3) * 16;           // 1024-output tile, first of its 16 lane slots
    const size_t ldq = (size_t)a.qtiles * (kQ4Tile / 2), lds = (size_t)a.qtiles * kQ4Tile;
    const uint8_t *codes = a.Mq + (size_t)tile * (kQ4Tile / 2) + (lb + i16) * 8;
    const uint16_t *xrow = ga.X + (size_t)min(tok0 + i16, batch - 1) * d_in;
    // the unit's outputs: tile * 1024 + h * 512 + lb * 8 + 0..127 for h = 0, 1
    const int col0 = tile * kQ4Tile + lb * 8;
    const int steps = d_in / kMfmaK, gsteps = 1 << (a.qshift - 5);     // groups hold 32 channels or more

    int lo, hi, w_lo, w_hi;
    balanced_share(steps, a.splits, split, lo, hi);
    balanced_share(hi - lo, kQ4Waves, w, w_lo, w_hi);
    w_lo += lo;
    w_hi += lo;

    f32x4 acc[16], grp[16], sx;                                 // [h * 8 + output] tiles: 4 outputs 8 r + ... of one token a lane
#pragma unroll
    for (int t = 0; t < 16; ++t) acc[t] = grp[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    sx = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint32_t one2 = DT == F16 ? 0x3c003c00u : 0x3f803f80u;
    const u32x4 ones = {one2, one2, one2, one2};
    uint16_t *s_sc = reinterpret_cast<uint16_t *>(smem + w * 768);
    uint8_t *s_zp = smem + w * 768 + 512;

    // scales and zero points of a group: lane l has outputs 4 l .. of the unit (128 per half h)
    u32x2 sc;
    uint32_t zp;
    auto request_group = [&](int g) {
        const size_t at = (size_t)min(g, (d_in >> a.qshift) - 1) * lds + col0 + (lane >> 5) * 512 + (lane & 31) * 4;
        sc = *reinterpret_cast<const u32x2 *>(a.qs + at);
        zp = *reinterpret_cast<const uint32_t *>(a.qz + at);
    };
    auto use_step = [&](const Q4Step &v, int s) {
        u32x4 b[1] = {v.x};
        switch (mode) {
        case kMaskNone: break;
        case kMaskOwn: mask_step<1, kMaskOwn>(b, kp, 0u); break;
        case kMaskOwn | kMaskSigned: mask_step<1, kMaskOwn | kMaskSigned>(b, kp, 0u); break;
        case kMaskUnion: if (batch <= 16) mask_step<1, kMaskUnion>(b, kp, 0u); break;
        default: if (batch <= 16) mask_step<1, kMaskUnion | kMaskSigned>(b, kp, 0u); break;
        }
        if ((mode & kMaskUnion) && batch > 16) {       // the other tile's tokens count too
            const u32x4 o = *reinterpret_cast<const u32x4 *>(ga.X + (size_t)min((tok0 ^ 16) + i16, batch - 1) * d_in + s * kMfmaK + g4 * 8);
            mask_union_two(b[0], o, kp, (mode & kMaskSigned) != 0);
        }
        sx = mfma16<DT>(ones, b[0], sx);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4 o[2];
            operands<DT, 0>(v.c, h, o);
            grp[h * 8 + 0] = mfma16<DT>(o[0], b[0], grp[h * 8 + 0]); grp[h * 8 + 4] = mfma16<DT>(o[1], b[0], grp[h * 8 + 4]);
            operands<DT, 1>(v.c, h, o);
            grp[h * 8 + 1] = mfma16<DT>(o[0], b[0], grp[h * 8 + 1]); grp[h * 8 + 5] = mfma16<DT>(o[1], b[0], grp[h * 8 + 5]);
            operands<DT, 2>(v.c, h, o);
            grp[h * 8 + 2] = mfma16<DT>(o[0], b[0], grp[h * 8 + 2]); grp[h * 8 + 6] = mfma16<DT>(o[1], b[0], grp[h * 8 + 6]);
            operands<DT, 3>(v.c, h, o);
            grp[h * 8 + 3] = mfma16<DT>(o[0], b[0], grp[h * 8 + 3]); grp[h * 8 + 7] = mfma16<DT>(o[1], b[0], grp[h * 8 + 7]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto fold = [&](int next_group) {
        *reinterpret_cast<u32x2 *>(s_sc + lane * 4) = sc;
        *reinterpret_cast<uint32_t *>(s_zp + lane * 4) = zp;
        __builtin_amdgcn_wave_barrier();
        request_group(next_group);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // row 4 g4 + r of the tiles: outputs 8 (4 g4 + r) + 0..7 of the half
                float sf[8];
                unpack8<DT>(*reinterpret_cast<const u32x4 *>(s_sc + h * 128 + (g4 * 4 + r) * 8), sf);
                const u32x2 z8 = *reinterpret_cast<const u32x2 *>(s_zp + h * 128 + (g4 * 4 + r) * 8);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float zf = (float)((z8[e >> 2] >> (8 * (e & 3))) & 0xffu);
                    acc[h * 8 + e][r] = __builtin_fmaf(sf[e], __builtin_fmaf(-zf, sx[r], grp[h * 8 + e][r]), acc[h * 8 + e][r]);
                }
            }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int t = 0; t < 16; ++t) grp[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        sx = f32x4{0.f, 0.f, 0.f, 0.f};
    };

    if (w_lo < w_hi) {
        Q4Step va, vb;
        int g = w_lo >> (a.qshift - 5);
        request_group(g);
        load_step(codes, ldq, xrow, lane, w_lo, va);
        for (int s = w_lo; s < w_hi; s += 2) {
            load_step(codes, ldq, xrow, lane, min(s + 1, w_hi - 1), vb);
            use_step(va, s);
            if (((s + 1) & (gsteps - 1)) == 0 || s + 1 >= w_hi) fold(++g);
            if (s + 1 >= w_hi) break;
            load_step(codes, ldq, xrow, lane, min(s + 2, w_hi - 1), va);
            use_step(vb, s + 1);
            if (((s + 2) & (gsteps - 1)) == 0 || s + 2 >= w_hi) fold(++g);
        }
    }

    // ---- the waves meet in LDS, one half of the outputs at a time: [wave][128 outputs][16 tokens]
    float *red = reinterpret_cast<float *>(smem);
    float *out = a.t.yc + (size_t)ttile * a.t.yc_rows * 16;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(w * 128 + (g4 * 4 + r) * 8 + e) * 16 + i16] = acc[h * 8 + e][r];
        __syncthreads();
        for (int i = tid; i < 128 * 16; i += 64 * kQ4Waves) {
            float s = red[i];
#pragma unroll
            for (int ww = 1; ww < kQ4Waves; ++ww) s += red[ww * 2048 + i];
            if (tok0 + (i & 15) < batch)                       // (the next launch clears what it reads, real tokens only)
                __hip_atomic_fetch_add(out + (size_t)(col0 + h * 512) * 16 + i, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

}  // namespace

hipError_t launch_mfma_q4(const LayerView *L, const MatrixView *M, int n, const void *X, int batch, bool dense, int cus, hipStream_t stream)
{
    if (n < 1 || n > kMaxGroupLayers || batch < 1 || batch > 32) return hipErrorInvalidValue;
    MfmaQ4Args a{};
    a.X = (const uint16_t *)X; a.d_in = L[0].d_in; a.batch = batch;
    const int tiles = (batch + 15) / 16;
    int t_blocks = 0, units = 0;
    for (int i = 0; i < n; ++i) {
        const LayerView &v = L[i];
        const MatrixView &m = M[i];
        if (!v.Mq || !v.qs || !v.qz || !m.yc || v.qshift < 5 || v.d_in % kMfmaK || v.d_in != a.d_in || v.dtype != L[0].dtype) return hipErrorInvalidValue;
        MfmaQ4Job &c = a.job[i];
        MfmaJob &j = c.t;
        c.Mq = v.Mq; c.qz = v.qz; c.qs = v.qs; c.qtiles = v.qtiles; c.qshift = v.qshift;
        c.units = (v.qtiles - 1) * 4 + std::min(4, (v.d_out - (v.qtiles - 1) * kQ4Tile + 127) / 128);
        units += c.units;
        j.yc = m.yc; j.yc_rows = m.yc_rows; j.rank = dense ? 0 : v.rank;
        j.mask_mode = dense ? kMaskNone : (v.batch_mask_mode == 1 ? kMaskUnion : kMaskOwn) | (v.keep_signed ? kMaskSigned : 0);
        j.kp = KeepPattern{(uint32_t)(uint16_t)m.keep_min * 0x10001u, (v.dtype == F16 ? 0x7c00u : 0x7f80u) * 0x10001u};
        j.SVt = m.SVt; j.t = (unsigned char *)m.t; j.t_acc = m.t_acc; j.t_flags = m.t_flags;
        if (j.rank > 0 && (!j.SVt || !j.t || !j.t_acc || !j.t_flags)) return hipErrorInvalidValue;
        j.t_blocks = (j.rank + 31) / 32 * 2;
        t_blocks += j.t_blocks;
    }
    // A compute unit holds two workgroups.  The aim is that the workgroups of t and of the codes together stay within those slots, where the
    // last of them would begin when the others end, and that no few units have twice the work of the others: one workgroup of codes per unit
    // (rounded down), or two where that is no fewer splits than twice as many and leaves a wave six steps or more (each split adds to every output;
    // between three and six the same).  us a pass, bf16, nearest to one workgroup per unit with t in four K slices -> this: gate, up and down of
    // 4096 / 11008 (two, rank 512; 264 + 256 workgroups -> 352 + 128) 119.4 at sixteen tokens -> 103.4, 164.8 at 32 -> 154.5, dense 114.2 ->
    // 100.2, 106.7 at four in fp16 -> 96.0; of 4096 / 14336 54.2 -> 52.9; one per unit alone 107.9, 165.0, 100.3, 98.8 and 54.2.  Two per unit with
    // shorter runs: 4096 x 4096 (eight, 16 splits) 112 -> 128, 2048 / 5632 (six) 185 -> 193.
    // A single split of 129 to 170 workgroups leaves a third of the units or more idle; there all that the slots hold, whatever the runs (two pairs
    // of layers, rank d_in / 16, 1 - 2 - 3 splits of 144: d_in 1024 39.9 - 40.8 - 39.1, 1536 50.2 - 50.5 - 43.4, 2048 60.2 - 57.4 - 52.0, 3072
    // 78.8 - 73.7 - 61.7).  And the nearest number to one per unit, a few units with two, where it makes runs of two steps out of three
    // (down - nearest: 44 a split, d_in 1536 30.2 - 28.5, 68, 1024 30.8 - 29.7, 52, 1280 30.2 - 28.6; but of three out of four 44, 2048 31.7 - 34.5).
    const int slots = 2 * cus, per_split = units * tiles, slices = mfma_t_slices(t_blocks, a.d_in, kQ4Waves, cus), steps = a.d_in / kMfmaK;
    const int one = cus / per_split, near = (cus + per_split / 2) / per_split, two = std::max(0, slots - t_blocks * std::min(2, slices)) / per_split;
    auto longest_run = [&](int k) { return ((steps + k - 1) / k + kQ4Waves - 1) / kQ4Waves; };
    const bool twice = two >= std::max(1, 2 * one) && (steps >= 6 * kQ4Waves * two || (one == 1 && two >= 3));
    const bool nearest = one > 0 && near > one && longest_run(one) == 3 && longest_run(near) == 2;
    const int splits = std::max(1, std::min(twice ? two : nearest ? near : one, steps / kQ4Waves));
    a.t_slices = t_blocks > 0 ? std::max(1, std::min(slices, (slots - per_split * splits) / t_blocks)) : 1;
    int t_total = 0, w_total = 0;
    for (int i = 0; i < kMaxGroupLayers; ++i) {
        if (i < n) {
            a.job[i].splits = splits;
            t_total += a.job[i].t.t_blocks * a.t_slices;
            w_total += a.job[i].units * a.job[i].splits * tiles;
        }
        a.t_end[i] = t_total;
        a.w_end[i] = w_total;
    }
    dim3 grid(t_total + w_total), block(64 * kQ4Waves);
    if (L[0].dtype == F16) {
        if (tiles == 1) hipLaunchKernelGGL((k_mfma_q4<F16, 1>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((k_mfma_q4<F16, 2>), grid, block, 0, stream, a);
    } else {
        if (tiles == 1) hipLaunchKernelGGL((k_mfma_q4<BF16, 1>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((k_mfma_q4<BF16, 2>), grid, block, 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace rsparse
