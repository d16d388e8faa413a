// Dense product Y = X W^T on the vector ALU, row-dot form, over the operand-layout copy of W (MatrixView::W: [block of 16
// rows][step of 32 columns][64 lanes][16 bytes], lane l = columns 8 (l / 16) .. + 7 of row l % 16).
//
// A workgroup of 8 waves owns 8 rows, half a block: a wave's load is the same 8 chunks of 8 columns of its rows, whole
// 128-byte lines, and wave w takes chunks 8 w .. + 7 of every 64, two loads to a batch and two batches in flight.  At one
// token a lane reads its chunk of x beside the weights (128 bytes per load, from cache), so that nothing is waited for before
// the weights are requested; with more tokens x is staged in LDS.  The 64 partial sums of a row (8 per wave) meet in LDS and
// wave w adds up those of row w.  No sum crosses workgroups: no atomics, no second launch.  Column chunk c belongs to partial
// sum c % 64 and is added in ascending order, and the 64 are added up by the butterfly of wave_sum, whatever the grid.
// Bound by HBM, below 2^23 weights by the launch and one chain of latencies.  Measured (us in a replayed graph over 512 MB of
// layers, fp16, one token; a row-major copy of W with a wave per row -> this): 1024 x 1024 3.30 -> 2.84, 2048 x 2048 4.91 ->
// 3.86, 4096 x 4096 7.5 -> 7.6, 8192 x 8192 22.5 -> 22.2.  16 rows and waves per workgroup: 3.17, 4.24, 7.6, 22.9.
#include "kernels.h"
#include "device_common.h"

#include <algorithm>

namespace rsparse {
namespace {

constexpr int kRows = 8, kChunks = 64 / kRows, kRowdotBatch = 2, kRowPitch = 65;

struct RowdotArgs {
    const uint16_t *W[kMaxGroupLayers];
    void *Y[kMaxGroupLayers];
    int d_out[kMaxGroupLayers], out_dtype[kMaxGroupLayers];
    int unit_end[kMaxGroupLayers];   // workgroups of layers 0..i
    const uint16_t *X;
    int batch, d_in;
};

template <int DT, int BT, bool NT>
__global__ __launch_bounds__(64 * kRows) void k_dense_rowdot(const RowdotArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr bool kDirect = BT == 1;
    const int tid = threadIdx.x, lane = tid & 63, w = uniform(tid >> 6);
    int job = 0, unit = (int)blockIdx.x;
#pragma unroll
    for (int j = 0; j < kMaxGroupLayers - 1; ++j)
        if ((int)blockIdx.x >= a.unit_end[j]) { job = j + 1; unit = (int)blockIdx.x - a.unit_end[j]; }
    const int d_in = a.d_in, nq = d_in / 8, steps = (d_in + 31) / 32;
    const int b0 = blockIdx.z * BT, nb = min(BT, a.batch - b0);
    const int row0 = unit * kRows, r = lane % kRows, cl = lane / kRows;
    const uint16_t *const mat = a.W[job] + ((size_t)(row0 / 16) * steps * 64 + row0 % 16 + r) * 8;
    const uint16_t *const x = a.X + (size_t)b0 * d_in;
    uint16_t *const s_x = reinterpret_cast<uint16_t *>(smem);  // [BT][d_in], zero past the batch

    struct Loads {
        u32x4 w[kRowdotBatch], x[kDirect ? kRowdotBatch : 1];
    } va, vb;
    // chunk q of my row: 16 bytes at [step q / 4][group q % 4]; zeros past the row
    auto load = [&](Loads &v, int p0) {
#pragma unroll
        for (int u = 0; u < kRowdotBatch; ++u) {
            const int q = (p0 + u * kRows) * kChunks + cl;
            v.w[u] = u32x4{0, 0, 0, 0};
            if constexpr (kDirect) v.x[u] = u32x4{0, 0, 0, 0};
            if (q < nq) {
                v.w[u] = ldg16<NT>(mat + (size_t)q * 128);
                if constexpr (kDirect) v.x[u] = *reinterpret_cast<const u32x4 *>(x + q * 8);
            }
        }
    };
    load(va, w);

    if constexpr (!kDirect) {
        for (int q = tid; q < nq; q += 64 * kRows)
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                u32x4 v = u32x4{0, 0, 0, 0};
                if (b < nb) v = *reinterpret_cast<const u32x4 *>(x + (size_t)b * d_in + q * 8);
                *reinterpret_cast<u32x4 *>(s_x + (size_t)b * d_in + q * 8) = v;
            }
        __syncthreads();
    }

    float acc[BT];
#pragma unroll
    for (int b = 0; b < BT; ++b) acc[b] = 0.f;
    auto use = [&](const Loads &v, int p0) {
#pragma unroll
        for (int u = 0; u < kRowdotBatch; ++u) {
            const int q = (p0 + u * kRows) * kChunks + cl;
            float f[8];
            unpack8<DT>(v.w[u], f);
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                u32x4 xq;
                if constexpr (kDirect) xq = v.x[u];
                else xq = q < nq ? *reinterpret_cast<const u32x4 *>(s_x + (size_t)b * d_in + q * 8) : u32x4{0, 0, 0, 0};
                float xf[8];
                unpack8<DT>(xq, xf);
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[b] = __builtin_fmaf(f[e], xf[e], acc[b]);
            }
        }
    };
    constexpr int kStep = kRows * kRowdotBatch;
    for (int p = w; p * kChunks < nq; p += 2 * kStep) {
        load(vb, p + kStep);
        use(va, p);
        load(va, p + 2 * kStep);
        use(vb, p + kStep);
    }
    if constexpr (!kDirect) __syncthreads();                   // the tokens are read: their LDS takes the partial sums
    float *const red = reinterpret_cast<float *>(smem);        // [BT][8 rows][64]
#pragma unroll
    for (int b = 0; b < BT; ++b) red[(b * kRows + r) * kRowPitch + w * kChunks + cl] = acc[b];
    __syncthreads();
    const int row = row0 + w;
#pragma unroll
    for (int b = 0; b < BT; ++b) {
        const float v = wave_sum(red[(b * kRows + w) * kRowPitch + lane]);
        if (lane == 0 && b < nb && row < a.d_out[job]) store_out(a.Y[job], (size_t)(b0 + b) * a.d_out[job] + row, v, a.out_dtype[job]);
    }
}

int rowdot_batch_tile(int batch) { return batch <= 1 ? 1 : batch <= 2 ? 2 : batch <= 4 ? 4 : 8; }

}  // namespace

bool rowdot_supported(int d_in, int batch) { return (size_t)rowdot_batch_tile(batch) * d_in * 2 <= 65536; }

hipError_t launch_dense_rowdot(const LayerView *L, const MatrixView *M, const Launch *cfg, int n, const void *X, int batch, void *const *Y,
                               hipStream_t stream)
{
    if (n < 1 || n > kMaxGroupLayers || batch < 1 || !rowdot_supported(L[0].d_in, batch)) return hipErrorInvalidValue;
    const int bt = rowdot_batch_tile(batch);
    RowdotArgs a{};
    a.X = (const uint16_t *)X; a.batch = batch; a.d_in = L[0].d_in;
    int total = 0;
    for (int i = 0; i < kMaxGroupLayers; ++i) {
        if (i < n) {
            if (!M[i].W || !Y[i] || L[i].d_in != a.d_in || L[i].dtype != L[0].dtype) return hipErrorInvalidValue;
            a.W[i] = M[i].W; a.Y[i] = Y[i]; a.d_out[i] = L[i].d_out; a.out_dtype[i] = L[i].out_dtype;
            total += (L[i].d_out + kRows - 1) / kRows;
        }
        a.unit_end[i] = total;
    }
    const size_t lds = std::max(bt > 1 ? (size_t)bt * a.d_in * 2 : 0, (size_t)bt * kRows * kRowPitch * 4);
    const dim3 grid(total, 1, (batch + bt - 1) / bt), block(64 * kRows);
    const bool nt = cfg[0].nontemporal != 0;
#define RS_RB(DT, BT)                                                                                 \
    do {                                                                                              \
        if (nt) hipLaunchKernelGGL((k_dense_rowdot<DT, BT, true>), grid, block, lds, stream, a);      \
        else hipLaunchKernelGGL((k_dense_rowdot<DT, BT, false>), grid, block, lds, stream, a);        \
    } while (0)
#define RS_R(DT)                                                                                      \
    do {                                                                                              \
        if (bt == 1) RS_RB(DT, 1); else if (bt == 2) RS_RB(DT, 2); else if (bt == 4) RS_RB(DT, 4); else RS_RB(DT, 8); \
    } while (0)
    if (L[0].dtype == F16) RS_R(F16); else RS_R(BF16);
#undef RS_R
#undef RS_RB
    return hipGetLastError();
}

}  // namespace rsparse
