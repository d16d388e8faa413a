// gfx950 matrix-core path of the R-Sparse linear layer (R-Sparse, Sec. 3.4) for 5 to 32 tokens, and of the dense product
// from 2 (1 on the largest), over a copy of W in operand layout (dense_rowmajor = 1).
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
// slice of a block splits the sums into two 16-bit halves (hi + lo, ~16 mantissa bits of the fp32 t, 22 in fp16) and stores
// them in operand layout with write-through stores, waits for these to be acknowledged and sets the block's flag.  A unit of
// W waits for the flags (bounded) when its rows are done and adds U_r t.  fp16 halves cannot hold |t| >= 65520: fp16 layers
// store t in fp32 beside them, and a step that meets an infinite half is multiplied from there with the fp32 MFMA.  The t buffer is read with ordinary loads: its
// lines are first touched in a launch by readers that have seen the flags, so no older copy of them is in a cache.
// Measured (us per call, before: a first launch with sums over K slices in fp32 atomics, a split launch and a finish
// launch): 8192 x 8192 r 1024 60.3 -> 41.7 at 32 tokens, 53.1 -> 34.7 at 8; 4096 x 4096 r 256 23.1 -> 14.6 at 8; dense
// 4096 -> 14336 (two) and back 93.1 -> 71.1 at 16.
#include "device_mfma.h"

#include <algorithm>

namespace rsparse {
namespace {

struct MfmaArgs {
    MfmaJob job[kMaxGroupLayers];
    int t_end[kMaxGroupLayers];  // t tasks (block, K slice) of jobs 0..i
    int w_end[kMaxGroupLayers];  // units of W of jobs 0..i
    const uint16_t *X;
    int n, batch, d_in, t_slices;
    int phases;                  // 1: t, 2: the units of W, 3: both in this launch (the units of W wait for t)
    int wait_polls, skip_stage1;
};

// SUMS: the W part was summed by an earlier launch (yc), and t is read in fp32: what is left is U_r t, the sum and the rounding.
template <int DT, int NB, int NF, bool SUMS>
__global__ __launch_bounds__(512, NF == 1 ? 4 : 3) void k_mfma_rows(const MfmaArgs ga)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, w = uniform(tid >> 6), nw = uniform(nthr >> 6);
    const int d_in = ga.d_in, batch = ga.batch;
    using B = Batch<NB, NF>;
    const int steps = (d_in + kMfmaK - 1) / kMfmaK, n_batches = (steps + B::S - 1) / B::S;
    const size_t block_bytes = (size_t)steps * 1024;
    const unsigned char *x = reinterpret_cast<const unsigned char *>(ga.X);
    // the first t_wgs workgroups take a (block, K slice) of t each and wait for nothing; the others a unit of W each
    const int t_wgs = SUMS ? 0 : ga.t_end[kMaxGroupLayers - 1] * (ga.phases & 1);
    const bool is_t = !SUMS && (int)blockIdx.x < t_wgs;
    const int first = is_t ? (int)blockIdx.x : (int)blockIdx.x - t_wgs;
    int job = 0, begin = 0;
#pragma unroll
    for (int j = 0; j < kMaxGroupLayers - 1; ++j) {
        const int e = is_t ? ga.t_end[j] : ga.w_end[j];
        if (first >= e) { job = j + 1; begin = e; }
    }
    const MfmaJob &jb = ga.job[job];
    if constexpr (!SUMS) {
        if (is_t) {
            t_unit<DT, NF, true>(jb, ga.X, batch, d_in, (first - begin) / ga.t_slices, (first - begin) % ga.t_slices, ga.t_slices, ga.phases == 3,
                                 ga.skip_stage1, smem);
            return;
        }
    }
    const KeepPattern kp = jb.kp;
    const int unit = first - begin, block0 = unit * NB, n_blocks = (jb.d_out + 15) / 16;
    // tokens past the batch repeat its last one; their results are not used
    uint32_t xoff[B::kX];
#pragma unroll
    for (int j = 0; j < B::kX; ++j) xoff[j] = (uint32_t)min(j * (64 / B::kLanes) + lane / B::kLanes, batch - 1) * (uint32_t)d_in * 2u;
    constexpr int kTiles = NB * NF;
    // a wave's LDS: its tokens' staging, and its D tiles when the waves meet
    constexpr int kWaveLds = NF * 16 * B::kPitch > kTiles * 1024 ? NF * 16 * B::kPitch : kTiles * 1024;
    unsigned char *sx = smem + (size_t)w * kWaveLds;

    const unsigned char *mat = reinterpret_cast<const unsigned char *>(jb.W) + (size_t)block0 * block_bytes;
    size_t aoff[NB];                                            // (blocks past the matrix: the last one again)
#pragma unroll
    for (int k = 0; k < NB; ++k) aoff[k] = (size_t)min(k, n_blocks - 1 - block0) * block_bytes;

    Batch<NB, NF> va;
    if constexpr (!SUMS) load_batch<NB, NF>(mat, aoff, x, xoff, lane, d_in, steps, w, va);

    // ---- which tokens keep a channel, for read-back: the last wave, 16 channels at a time (a lane = a token)
    if (w == nw - 1) {
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
#define RS_STREAM(MODE) stream_rows<DT, NB, NF, MODE>(mat, aoff, x, xoff, sx, kp, 0u, lane, d_in, w, n_batches, nw, va, acc)
    if constexpr (!SUMS) {
        switch (jb.mask_mode) {
        case kMaskNone: RS_STREAM(kMaskNone); break;
        case kMaskOwn: RS_STREAM(kMaskOwn); break;
        case kMaskUnion: RS_STREAM(kMaskUnion); break;
        case kMaskOwn | kMaskSigned: RS_STREAM(kMaskOwn | kMaskSigned); break;
        default: RS_STREAM(kMaskUnion | kMaskSigned); break;
        }
    }
#undef RS_STREAM
    const bool lowrank = jb.t_blocks > 0, hand_off = lowrank && !SUMS && ga.phases == 3;

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

    // ---- U_r t: the rank's steps of 32, one per wave in turn; the rows of U_r are requested before t is waited for
    if (lowrank) {
        f32x4 ah[2][NB][NF];                                   // the products with t's parts (SUMS: with t, the first alone)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int f = 0; f < NF; ++f) ah[h][i][f] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int usteps = (jb.rank + kMfmaK - 1) / kMfmaK;
        const size_t ublock = (size_t)usteps * 1024;
        const unsigned char *um = reinterpret_cast<const unsigned char *>(jb.U) + (size_t)block0 * ublock + lane * 16;
        // (steps whose loads are requested together; t comes from L2 and nothing else hides its latency)
        constexpr int US = SUMS || NB * NF == 1 ? 4 : 2;
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
        auto t_as_it_is = [&](int s, int f, f32x4 (&tf)[2]) {
            const float *p = jb.t32() + ((size_t)(s * NF + f) * 64 + lane) * 8;
            tf[0] = *reinterpret_cast<const f32x4 *>(p);
            tf[1] = *reinterpret_cast<const f32x4 *>(p + 4);
        };
        for (int s0 = w; s0 < usteps; s0 += nw * US) {
            if constexpr (SUMS) {
                f32x4 tf[US][NF][2];
#pragma unroll
                for (int u = 0; u < US; ++u)
#pragma unroll
                    for (int f = 0; f < NF; ++f) t_as_it_is(min(s0 + u * nw, usteps - 1), f, tf[u][f]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < US; ++u) {
                    if (s0 + u * nw < usteps) {
#pragma unroll
                        for (int i = 0; i < NB; ++i)
#pragma unroll
                            for (int f = 0; f < NF; ++f) ah[0][i][f] = mfma_f32<DT>(ua[u][i], tf[u][f], ah[0][i][f]);
                    }
                }
            } else {
                u32x4 th[US][NF][2];
                uint32_t beyond = 0u;                          // fp16: sign bits where a first part is infinite or NaN
#pragma unroll
                for (int u = 0; u < US; ++u) {
                    const int s = min(s0 + u * nw, usteps - 1);
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        const unsigned char *p = jb.t + (size_t)(s * NF + f) * 2048 + lane * 16;
#pragma unroll
                        for (int h = 0; h < 2; ++h) th[u][f][h] = *reinterpret_cast<const u32x4 *>(p + h * 1024);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (DT == F16) {
#pragma unroll
                    for (int u = 0; u < US; ++u)
#pragma unroll
                        for (int f = 0; f < NF; ++f)
#pragma unroll
                            for (int e = 0; e < 4; ++e) beyond |= (th[u][f][0][e] & 0x7c007c00u) + 0x04000400u;
                }
                if (DT == F16 && __any((beyond & 0x80008000u) != 0u)) {
                    // some t is beyond fp16's range: these steps in fp32
                    for (int u = 0; u < US && s0 + u * nw < usteps; ++u) {
                        u32x4 au[NB];
#pragma unroll
                        for (int i = 0; i < NB; ++i)
                            au[i] = ld16(um + min(i, n_blocks - 1 - block0) * ublock + (size_t)(s0 + u * nw) * 1024);
#pragma unroll
                        for (int f = 0; f < NF; ++f) {
                            f32x4 tf[2];
                            t_as_it_is(s0 + u * nw, f, tf);
#pragma unroll
                            for (int i = 0; i < NB; ++i) ah[0][i][f] = mfma_f32<DT>(au[i], tf, ah[0][i][f]);
                        }
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < US; ++u) {
                        if (s0 + u * nw < usteps) {
#pragma unroll
                            for (int i = 0; i < NB; ++i)
#pragma unroll
                                for (int f = 0; f < NF; ++f)
#pragma unroll
                                    for (int h = 0; h < 2; ++h) ah[h][i][f] = mfma16<DT>(ua[u][i], th[u][f][h], ah[h][i][f]);
                        }
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
                for (int j = 0; j < 4; ++j) acc[i][f][j] += SUMS ? ah[0][i][f][j] : ah[0][i][f][j] + ah[1][i][f][j] * (1.0f / LoScale<DT>::value);
    }

    meet();
    // every wave of this workgroup has read t: count the unit, over kTReadSubs counters first, so that the units, which end
    // together, do not queue up on one address (the answer is looked at after the stores)
    const bool counted = hand_off && tid == 0;
    const int sub = unit % kTReadSubs;
    int *const t_read = jb.t_flags + t_read_at(jb.rank);
    int arrived = -1;
    if (counted) arrived = __hip_atomic_fetch_add(t_read + sub * 32, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int item = tid; item < kTiles * 64; item += nthr) {
        const int l = item & 63, tile = item >> 6, i = tile / NF, f = tile % NF;
        f32x4 s = sum_up(item);
        const int tok = f * 16 + (l & 15);
        const int row = (block0 + i) * 16 + 4 * (l >> 4);       // four consecutive rows (d_out is a multiple of 8)
        if (tok < batch && row < jb.d_out) {
            if constexpr (SUMS) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float *y = jb.yc + ((size_t)f * jb.yc_rows + row + j) * 16 + (l & 15);
                    s[j] += *y;
                    *y = 0.f;
                }
            }
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

size_t mfma_t_bytes(int rank) { return t32_offset(rank) * 2; }

// 64 x 64 tiles through LDS, 16 bytes per access on both sides.
__global__ __launch_bounds__(256) void k_transpose16(const uint16_t *src, size_t rows, size_t cols, uint16_t *dst, size_t ld)
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
            *reinterpret_cast<u32x4 *>(dst + c * ld + r) = v;
        }
    }
}

hipError_t launch_transpose16(const uint16_t *src, size_t rows, size_t cols, uint16_t *dst, size_t ld, hipStream_t stream)
{
    if (rows == 0 || cols == 0) return hipSuccess;
    hipLaunchKernelGGL(k_transpose16, dim3((unsigned)((cols + 63) / 64), (unsigned)((rows + 63) / 64)), dim3(256), 0, stream, src, rows, cols, dst, ld);
    return hipGetLastError();
}

// K slices of t: enough workgroups for the chip, a batch of loads for every wave of nw, and at most four, whose sums meet in
// atomics (8192 x 8192, rank 1024, 8 tokens: 43.5 us with one slice, 39.0 with two, 34.5 with four; 4096 x 4096, rank 256:
// 16.1 with one, 14.6 with four, 15.4 with sixteen)
int mfma_t_slices(int t_blocks, int d_in, int nw, int cus)
{
    return t_blocks > 0 ? std::max(1, std::min({4, cus / t_blocks, (d_in + kMfmaK * 4 - 1) / (kMfmaK * 4) / nw})) : 1;
}

hipError_t launch_mfma(const LayerView *L, const MatrixView *M, int n, const void *X, int batch, void *const *Y, uint32_t *const *chan_bits, int cus,
                       int phases, bool dense, int wait_polls, int skip_stage1, hipStream_t stream)
{
    if (n < 1 || n > kMaxGroupLayers || batch < 1 || batch > 32 || phases < 1 || phases > 3 || (!M[0].W && phases != 2)) return hipErrorInvalidValue;
    const int nf = batch > 16 ? 2 : 1;
    MfmaArgs a{};
    a.n = n; a.X = (const uint16_t *)X; a.batch = batch; a.d_in = L[0].d_in; a.phases = phases;
    a.wait_polls = wait_polls > 0 ? wait_polls : kWaitLimitPolls;
    a.skip_stage1 = skip_stage1;
    // Where the W part was summed by an earlier launch t stays in 32 bits, as those layers' vector kernels keep it; beside a W part
    // it is multiplied in two 16-bit parts (fp16: 22 bits, in fp32 beyond its range; bf16: 16).  The fp32 MFMA has a sixteenth of
    // the rate: against parts in 16 bits 3 to 5 % of a call at 17 to 32 tokens (gate, up and down at 4096 / 11008, rank 512, fp16,
    // column-major 90.6 -> 94.8 us, 4-bit 72.0 -> 75.5) and at rank 1024 (8192 x 8192 at five tokens 35.6 -> 36.4), nothing else;
    // three exact 16-bit parts measured 94.4 to 98.4 and 75.7.
    const bool sums = M[0].W == nullptr;
    // Units of one block for up to 16 tokens, of two for more (a unit reads all tokens, from L2, beside its rows: at 32
    // tokens and one block twice the bytes of the rows; measured at 8192 x 8192, 32 tokens: dense 33.7 us with one block,
    // 27.0 with two; at 8 tokens 23.2 and 22.9, at 4096 -> 14336 with 16 tokens 70.9 and 78.1).  Four waves a unit: with eight
    // the same bytes are in flight in half the workgroups (8192 x 8192, 8 tokens: 24.7 against 25.8 us).  Without rows of W a unit
    // is one block at any batch (column-major 2048 x 2048, rank 256, 32 tokens: 15.5 us with two, 14.5 with one; gate, up and
    // down at 2048 / 5632, 24 tokens 47.4 and 45.4; alike at 4096 and 8192 channels).
    const int nb = sums ? 1 : nf, nw = 4;
    int w_total = 0, t_blocks = 0;
    for (int i = 0; i < n; ++i) {
        MfmaJob &jb = a.job[i];
        const LayerView &v = L[i];
        const MatrixView &m = M[i];
        if (v.d_in != a.d_in || v.dtype != L[0].dtype || (sums ? m.W || !m.yc : !m.W) || !Y[i]) return hipErrorInvalidValue;
        jb.W = m.W; jb.SVt = m.SVt; jb.U = m.U; jb.t = (unsigned char *)m.t; jb.Y = Y[i]; jb.bias = v.bias;
        jb.yc = m.yc; jb.yc_rows = m.yc_rows;
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
    const int batch_k = kMfmaK * (nf == 1 ? 4 : 2);
    a.t_slices = mfma_t_slices(t_blocks, a.d_in, nw, cus);
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
#define RS_M(DT, NB, NF, SV) hipLaunchKernelGGL((k_mfma_rows<DT, NB, NF, SV>), grid, block, lds, stream, a)
#define RS_MS(DT) do { if (nf == 1) { if (sums) RS_M(DT, 1, 1, true); else RS_M(DT, 1, 1, false); }    \
                       else { if (sums) RS_M(DT, 1, 2, true); else RS_M(DT, 2, 2, false); } } while (0)
    if (L[0].dtype == F16) RS_MS(F16); else RS_MS(BF16);
#undef RS_MS
#undef RS_M
    return hipGetLastError();
}

}  // namespace rsparse
