// gfx950 (MI355X, CDNA4) kernels of the R-Sparse linear layer (R-Sparse, Sec. 3.4).
//
// Everything here is bound by HBM bandwidth at decode batch sizes (2*B flops per 2-byte
// weight), so the kernels are organised around the weight stream: 16-byte loads, one
// 1 KiB row segment per 64-lane wave, many rows in flight, fp32 accumulation on the
// vector ALU.  Storage:
//
//   M    [d_in + r][d_out]  W column-major (row c = all outputs of input channel c; Sec. 3.4 asks
//                        for this layout so that a kept channel is one contiguous run), followed by
//                        U_r^T (row d_in + j = U_r[:, j]) for the one-launch kernel
//   SVt  [r][d_in]       S_r V_r^T, one singular component per row
//   SVc  [d_in][r]       optional channel-major copy of S_r V_r^T (row c = its column c): at one token the stage 1 of
//                        the one-launch kernel then reads the rows of the dropped channels only (stage1_gather)
//   U    [d_out][r]      U_r row-major
//
// One call is either two launches, ordered by the stream (no intra-kernel cross-workgroup waits):
//
//   k_sparse_and_t   workgroups [0, lr_wgs):  t_i = SVt[i,:] . (x - sigma_t(x))      (row dots)
//                    the others:              yacc += sum_{c kept} x_c M[c,:]         (gather-axpy)
//                    Each gather workgroup thresholds and compacts x itself (it scans the whole
//                    token -- 2*d_in bytes from L2 -- and keeps its balanced share of the ascending
//                    kept list), so there is no compaction launch.  Column tiles x channel splits
//                    fill the chip; partial sums meet in fp32 atomics.
//   k_finish         Y = round(yacc + U t)   (row dots over U, no reduction), yacc re-zeroed.
//
// or ONE launch (k_rsparse_fused), which removes the second kernel's launch and start-up latency:
// M carries r more rows, U_r^T, so that stage 2 of the low-rank part is r more "channels" whose
// coefficients are t.  Every gather wave ends with its share of those rows; only the FMAs of those rows need t,
// which the stage-1 workgroups (at the front of the grid, so dispatched first) publish as {tag, fp32 bits} (device_stage1.h).
// All cross-workgroup data (t, yacc, arrival counters) moves through agent-scope relaxed atomics, which are performed at the
// device's coherence point, so no cache write-back or invalidate is needed; a workgroup waits for its own atomics to be
// acknowledged (s_waitcnt) before it bumps a counter.  The last workgroup to arrive at a column tile swaps the
// tile's sums out of yacc (which re-zeroes them), rounds once and stores Y.  For the gate / up pair of an MLP (Sec. 3.1) the two
// layers share one set of counters and the finisher stores H = round(silu(g) * u) instead of g and u.
#include "kernels.h"
#include "device_common.h"
#include "device_gather.h"

#include <algorithm>

namespace rsparse {
#if RSPARSE_STAMPS
hipError_t set_stamp_buffer_columns(void *buf, int capacity_waves) { return set_stamps_of_this_file(buf, capacity_waves); }
#endif
namespace {

// ---------------------------------------------------------------------------------------------
// Streaming primitive: acc[b][0:8] += sum_j coef[j][b] * M[idx[j], col:col+8] over the n staged rows.
// Wave w of nw takes R consecutive rows per batch; a batch's loads are all issued before its
// first FMA, and the next batch is issued before the current one is consumed (two batches of
// 16-byte loads in flight per lane).  idx / coef live in LDS and are wave-uniform (scalar registers).
// ---------------------------------------------------------------------------------------------
template <bool NT, int R>
__device__ __forceinline__ void load_batch(const uint16_t *__restrict__ M, size_t ld, int col, bool colok,
                                           const int *s_idx, int n, int j0, u32x4 (&v)[R])
{
    if (j0 + R <= n) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const int idx = uniform(s_idx[j0 + u]);
            v[u] = colok ? ldg16<NT>(M + (size_t)idx * ld + col) : u32x4{0, 0, 0, 0};
        }
    } else {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            v[u] = u32x4{0, 0, 0, 0};
            if (j0 + u < n) {
                const int idx = uniform(s_idx[j0 + u]);
                if (colok) v[u] = ldg16<NT>(M + (size_t)idx * ld + col);
            }
        }
    }
}

template <int DT, int BT, int R>
__device__ __forceinline__ void fma_batch(const u32x4 (&v)[R], const float *s_coef, int n, int j0,
                                          float (&acc)[BT][8])
{
#pragma unroll
    for (int u = 0; u < R; ++u) {
        if (j0 + u < n) {
            float f[8];
            unpack8<DT>(v[u], f);
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                const float cf = uniform(s_coef[(j0 + u) * BT + b]);
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[b][e] = __builtin_fmaf(cf, f[e], acc[b][e]);
            }
        }
    }
}

// Consume the already-issued batch `va` (rows j0..) and stream the rest of the wave's rows.
// before_fma(j0) runs ahead of the FMAs of the batch that starts at row j0 (its loads, and those of
// the following batch, are already in flight).
template <int DT, int BT, bool NT, int R, typename Hook>
__device__ __forceinline__ void stream_rest(const uint16_t *__restrict__ M, size_t ld, int col, bool colok,
                                            const int *s_idx, const float *s_coef, int n, int j0, int step,
                                            u32x4 (&va)[R], float (&acc)[BT][8], Hook &&before_fma)
{
    u32x4 vb[R];
    while (j0 < n) {
        load_batch<NT, R>(M, ld, col, colok, s_idx, n, j0 + step, vb);
        before_fma(j0);
        fma_batch<DT, BT, R>(va, s_coef, n, j0, acc);
        j0 += step;
        if (j0 >= n) break;
        load_batch<NT, R>(M, ld, col, colok, s_idx, n, j0 + step, va);
        before_fma(j0);
        fma_batch<DT, BT, R>(vb, s_coef, n, j0, acc);
        j0 += step;
    }
}

// Cross-wave reduction of a column tile through LDS, then fp32 atomics into yacc.  No fences: in the
// two-launch form the kernel boundary before k_finish orders the atomics, in the one-launch form the
// caller waits for their acknowledgement (an agent-scope fence per workgroup costs an L2 write-back +
// invalidate on this chip and dominated the run time).
template <int BT>
__device__ __forceinline__ void reduce_to_yacc(float (&acc)[BT][8], float *s_red, float *yacc, int b0, int nb,
                                               int d_out, int tile)
{
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, w = tid >> 6, nw = nthr >> 6;
    const int colbase = tile * kTile;
    // b must stay a compile-time index: a run-time subscript would push acc[][] into scratch memory
#pragma unroll
    for (int b = 0; b < BT; ++b) {
        if (b >= nb) break;
        float *yrow = yacc + (size_t)(b0 + b) * d_out;
        if (nw > 1) {
            if (b > 0) __syncthreads();
            float4 *dst = reinterpret_cast<float4 *>(s_red + w * kTile + lane * 8);
            dst[0] = float4{acc[b][0], acc[b][1], acc[b][2], acc[b][3]};
            dst[1] = float4{acc[b][4], acc[b][5], acc[b][6], acc[b][7]};
            __syncthreads();
            for (int col = tid; col < kTile; col += nthr) {
                float s = 0.f;
                for (int i = 0; i < nw; ++i) s += s_red[i * kTile + col];
                if (colbase + col < d_out)
                    __hip_atomic_fetch_add(yrow + colbase + col, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int col = lane * 8 + e;
                if (colbase + col < d_out)
                    __hip_atomic_fetch_add(yrow + colbase + col, acc[b][e], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

// (what every workgroup reads first lies first)
struct GatherArgs {
    const uint16_t *X;
    int batch, splits, tiles, cap;
    int lr_wgs, lr_rows, lr_chunk;     // stage-1 workgroups at the front of the grid, rows each, LDS chunk
    int tile_map;
    int dense;                         // 4-bit kernels only: keep every channel (the dense baseline)
    LayerView L;
};

// What a gather workgroup of the one-launch kernel needs, side by side: it is fetched in a few wide scalar loads, and all of it
// before anything else (left alone, the compiler fetches an argument where it is used, a round trip each).
struct DirectArgs {
    const uint16_t *X, *M;
    const uint16_t *SVc;               // stage 1 over the channel-major copy of S_r V_r^T (stage1_gather), or null
    int *sync;
    unsigned long long *t_tag;
    float *yacc;
    uint32_t *act_bits;
    int d_in, d_out, rank, batch;
    int tiles, splits, cap, lr_wgs;
    uint32_t tiles_inv;                // 2^32 / tiles + 1 (0: one tile): g / tiles = umulhi(g, tiles_inv)
    int tile_map, union_all;
    float tau_ge;
    int q_base, q_rem, u_base, u_rem;  // balanced shares of d_in / 8 over the splits * waves waves of a tile, and of the rank over the splits
    int waves;                         // per workgroup
    int cap_s1;                        // list slots of a wave of stage1_gather
    int wait_polls;                    // bound on re-reads of a t entry that is not there yet
    void *Y;                           // the output, [batch][d_out]
    Stage1Args s1;
    LayerView L;
};

// Workgroup index -> (column tile, channel split).  Plain: tile-fastest.  XCD-aware: workgroups are
// handed to the 8 XCDs round-robin by index, and fp32 atomics from different XCDs to one line move
// it between their L2s; giving every split of a tile an index congruent to (tile mod 8) keeps a
// tile's accumulators in one L2.  Indices past the last real pair are idle.
__device__ __forceinline__ bool map_tile(int tile_map, int tiles, int splits, int g, int &tile, int &split)
{
    if (tile_map != 2) {
        tile = g % tiles;
        split = g / tiles;
        return true;
    }
    const int x = g & 7, slot = g >> 3;              // slot enumerates (tile / 8, split)
    const int tgroup = slot / splits;
    split = slot % splits;
    tile = tgroup * 8 + x;
    return tile < tiles;
}
__device__ __forceinline__ bool map_tile(const GatherArgs &a, int g, int &tile, int &split)
{
    return map_tile(a.tile_map, a.tiles, a.splits, g, tile, split);
}

struct GroupArgs {
    int wg_end[kMaxGroup];
    int n;
    GatherArgs job[kMaxGroup];
};
struct DirectGroupArgs {
    DirectArgs job[kMaxGroup];
    int wg_end[kMaxGroup];
    int n;
    int gate_up;       // jobs 0 and 1 are the gate and up projections of an MLP (same d_out);
                       // the column tiles are finished jointly and H = round(silu(g) * u) is stored to job[0].Y
};
// ---------------------------------------------------------------------------------------------
// The one-launch kernel (16-bit weights).  What bounds a call of a decoder's size is not the stream but the chain of dependent
// round trips to memory (0.9 us each) around it: token -> rows -> sums -> arrival -> swap, and the same for t before its last
// rows.  So a wave owns fixed chunks of 8 channels (chunk rho, rho + R, ... of the R = splits * waves waves of the column
// tile: neighbouring channels go to different waves, whatever part of the token is large), reads only those channels of
// the token(s), thresholds them (Sec. 3.4, sigma_t) and compacts the kept ones with ballots into the workgroup's list in LDS: no scan of
// the whole token and one barrier in front of the first weight load, and little code, which runs once per launch from a
// cold instruction cache.  After the barrier the waves claim batches of the list and of the split's rows of U_r^T (SharedRows).
// Rows are read through a buffer descriptor: a lane past the last column or a list entry past the list's end lies outside of it
// and reads zero without touching memory, so that every load is unconditional and the compiler counts the outstanding ones
// exactly.  Measured, a scan of the whole token and one balanced list of all splits per workgroup -> this (us per pass, one token):
// 4096 x 4096 10.8 -> 9.3, gate / up and down at 4096 / 11008 (four) 172.7 -> 171.0, an 8192 / 28672 block 206.9 -> 202.1, with a fixed count
// 5128 / 13832 (two) 146.7 -> 138.4; four tokens at 4096 / 14336 (two) 162.9 -> 154.3.  Equal shares of the list -> claimed batches, with
// the rows form of stage 1 in a kernel of its own (one token: 62 or 63 registers, three workgroups to a compute unit, for 94 and two): 9.3 ->
// 9.05, 167 -> 158.7, 201.5 -> 197.0, 136.5 -> 133.4; 154.8 -> 147.0.
// ---------------------------------------------------------------------------------------------
// What a wave compacts: chunk j of its n_ch chunks holds channels ((j * step + first) * 8 ..) + 7.
template <int BT>
struct Channels {
    const uint16_t *X;
    int d_in, batch, b0, nb, n_ch, step, first;
    bool union_all;
    TileRules<BT> rules;
};
template <int BT> constexpr int kTokenPieces = BT == 1 ? 3 : BT == 2 ? 2 : 1;     // runs of 64 channels requested together

template <int BT>
__device__ __forceinline__ void request_channels(const Channels<BT> &ch, int p0, uint32_t (&xr)[kTokenPieces<BT>][BT])
{
    const int lane = threadIdx.x & 63;
    const __amdgpu_buffer_rsrc_t tokens = buffer_of(ch.X, (uint32_t)ch.batch * ch.d_in * 2u);
#pragma unroll
    for (int j = 0; j < kTokenPieces<BT>; ++j) {
        const int jc = (p0 + j) * 8 + (lane >> 3), c = (jc * ch.step + ch.first) * 8 + (lane & 7);
        // (past my channels or the batch: outside, zero)
#pragma unroll
        for (int b = 0; b < BT; ++b)
            xr[j][b] = __builtin_amdgcn_raw_buffer_load_b16(tokens, (int)(jc < ch.n_ch && b < ch.nb ? (uint32_t)((ch.b0 + b) * ch.d_in + c) * 2u : kOutside), 0, 0);
    }
}

// The channels that some token keeps (DROP: drops), appended to the workgroup's list: offsets c * pitch of their rows in s_off, the
// coefficients of the tile's tokens in s_cf [entry][BT].  One lane per channel: the channels of a ballot, their places a count of the
// lower lanes' bits, and one addition to the list's length *s_n (LDS) for the wave's run of channels.  The first channels have been
// requested.  act_bits (or null): which tokens keep each channel, for read-back.
template <int DT, int BT, bool EXT, bool DROP>
__device__ __forceinline__ void compact_channels(const Channels<BT> &ch, const LayerView &L, uint32_t pitch, uint32_t (&xr)[kTokenPieces<BT>][BT],
                                                 uint32_t *s_off, uint32_t *s_cf, int *s_n, uint32_t *act_bits)
{
    constexpr int PX = kTokenPieces<BT>;
    const int lane = threadIdx.x & 63, np = (ch.n_ch + 7) >> 3;
    for (int p0 = 0; p0 < np; p0 += PX) {
        if (p0 > 0) request_channels<BT>(ch, p0, xr);
        unsigned long long mask[PX];
        uint32_t listed[PX];                 // bit b: token b has a coefficient on the lane's channel
        int n = 0;
#pragma unroll
        for (int j = 0; j < PX; ++j) {
            const int jc = (p0 + j) * 8 + (lane >> 3), c = (jc * ch.step + ch.first) * 8 + (lane & 7);
            const bool valid = jc < ch.n_ch;
            bool kb[BT], any = false;
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                const float xf = widen16<DT>((uint16_t)xr[j][b]);
                kb[b] = valid && b < ch.nb && (EXT ? keep(xf, c, ch.rules.r[b], ch.rules.sgn) : keep_threshold(xf, ch.rules.r[b]));
                any = any || kb[b];
            }
            if (BT > 1 && ch.union_all) {
                // every token uses the union over the WHOLE batch (also the tokens of other batch tiles)
                for (int bb = 0; bb < ch.batch; ++bb) {
                    if (bb >= ch.b0 && bb < ch.b0 + ch.nb) continue;
                    const float xo = valid ? widen16<DT>(as_global(ch.X)[(size_t)bb * ch.d_in + c]) : 0.f;
                    any = any || (valid && keep(xo, c, EXT ? rule_of(L, bb) : ch.rules.r[0], ch.rules.sgn));
                }
#pragma unroll
                for (int b = 0; b < BT; ++b) kb[b] = any && b < ch.nb;
            }
            uint32_t bits = 0;
#pragma unroll
            for (int b = 0; b < BT; ++b) bits |= (uint32_t)kb[b] << b;
            if (!DROP && act_bits && valid) act_bits[c] = bits;
            if (DROP) {
                bits = valid ? ~bits & ((1u << ch.nb) - 1u) : 0u;
                any = bits != 0u;
            }
            listed[j] = bits;
            mask[j] = __ballot(any);
            n += __popcll(mask[j]);
        }
        if (n == 0) continue;
        int at = 0;
        if (lane == 0) at = __hip_atomic_fetch_add(s_n, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        at = uniform(at);
#pragma unroll
        for (int j = 0; j < PX; ++j) {
            const int c = (((p0 + j) * 8 + (lane >> 3)) * ch.step + ch.first) * 8 + (lane & 7);
            const int e = at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask[j], 0u));
            if ((mask[j] >> lane) & 1u) {
                s_off[e] = (uint32_t)c * pitch;
#pragma unroll
                for (int b = 0; b < BT; ++b) s_cf[e * BT + b] = (listed[j] >> b) & 1u ? as_u(widen16<DT>((uint16_t)xr[j][b])) : 0u;
            }
            at += __popcll(mask[j]);
        }
    }
}

// What the waves of a workgroup (or those of one column part) stream together: the n entries of the list and behind them, to n_all,
// n_all - n rows at extra_off, + pitch, ...  They take it in batches: the first two of a wave are its own, the others are
// claimed at *s_next (LDS) one batch ahead.  A compute unit serves the waves of its lower slots first: with equal shares for the waves the
// first of a workgroup ended at 62 us and the last at 91 (8192 -> 28672, two layers, one token), and what is left of the memory
// system's queue at the end of a launch is too short to fill it.
struct SharedRows {
    const uint32_t *off, *cf;            // [n], [n][BT]
    int n, n_all, first, second, *s_next;
    uint32_t extra_off, pitch;
};

// acc[b][0:8] += sum_i cf_i[b] row_i[lane_off ..] over the batches of R rows that the wave gets, two in flight.  Lane u holds entry u of
// a batch; its row offset and coefficients become wave-uniform with one readlane each.  extra(i, lane has one, q): the
// coefficients of the rows behind the list, as {., bits}; settle: ahead of the products of a batch that holds some.
template <int DT, int BT, bool NT, int R, typename Extra, typename Settle>
__device__ __forceinline__ int stream_rows(__amdgpu_buffer_rsrc_t rows, uint32_t lane_off, const SharedRows &sr, float (&acc)[BT][8], Extra &&extra, Settle &&settle)
{
    const int lane = threadIdx.x & 63, n = sr.n, n_all = sr.n_all, last = max(n - 1, 0);
    struct Batch {
        int at;
        u32x4 v[R];
        unsigned long long q[BT];
    };
    auto row_offsets = [&](int at) {
        const int e = at + lane;
        const uint32_t listed = sr.off[min(e, last)];
        return lane >= R || e >= n_all ? kRowOutside : e < n ? listed : sr.extra_off + (uint32_t)(e - n) * sr.pitch;
    };
    auto claim = [&]() {
        int c = 0;
        if (lane == 0) c = __hip_atomic_fetch_add(sr.s_next, R, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return c;
    };
    auto issue = [&](Batch &q, int at, uint32_t ov) {
        q.at = at;
#pragma unroll
        for (int u = 0; u < R; ++u) q.v[u] = buffer_load16<NT>(rows, lane_off + lane_value(ov, u));
        __builtin_amdgcn_sched_barrier(0);
        const int e = at + lane;
#pragma unroll
        for (int b = 0; b < BT; ++b) q.q[b] = e < n ? (unsigned long long)sr.cf[min(e, last) * BT + b] : 0ull;
        if (at + R > n && at < n_all) extra(e - n, lane < R && e >= n && e < n_all, q.q);
    };
    auto consume = [&](Batch &q) {
        if (q.at + R > n && q.at < n_all) settle(q.at + lane - n, lane < R && q.at + lane >= n && q.at + lane < n_all, q.q);
#pragma unroll
        for (int u = 0; u < R; ++u) {
            float f[8];
            unpack8<DT>(q.v[u], f);
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                const float cf = as_f(lane_value((uint32_t)q.q[b], u));
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[b][e] = __builtin_fmaf(cf, f[e], acc[b][e]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int done = 0;                        // (rows, for the time stamps)
    Batch qa, qb;
    uint32_t ov = row_offsets(sr.first);
    int next = sr.second, c = claim();
    issue(qa, sr.first, ov);
    ov = row_offsets(next);
    for (;;) {
        issue(qb, next, ov);
        next = uniform(c);
        ov = row_offsets(next);
        c = claim();
        consume(qa);
        done += max(0, min(R, n_all - qa.at));
        if (qb.at >= n_all) break;
        issue(qa, next, ov);
        next = uniform(c);
        ov = row_offsets(next);
        c = claim();
        consume(qb);
        done += max(0, min(R, n_all - qb.at));
        if (qa.at >= n_all) break;
    }
    return done;
}

// Stage 1 of the low-rank part over the channel-major copy SVc [d_in][rank] (row c = (S_r V_r^T)[:, c]), up to four tokens:
// t = sum over the DROPPED channels c of x_c SVc[c, :] (Sec. 3.4: the low-rank part acts on x - sigma_t(x), whose kept
// channels are zero), so only the rows of dropped channels are read -- rank * (d_in - k) elements instead of rank * d_in.  A wave
// takes 512 columns (part w % parts) of the rows of its own channels, the waves of a part meet in LDS, and the workgroup's
// partial t goes to t_sum with fp32 atomics.  The last workgroup to arrive swaps the sums out (which re-zeroes them) and
// publishes t.  No workgroup waits for another here.
template <int DT, int BT, bool NT, bool EXT, int R>
__device__ __forceinline__ void stage1_gather(const DirectArgs &h, const LayerView &L, unsigned char *smem, int wg, int z)
{
    RS_STAMP_DECL;
    RS_STAMP(1);
    const int tid = threadIdx.x, lane = tid & 63, w = uniform(tid >> 6), nw = h.waves, nthr = nw * 64;
    const int d_in = h.d_in, r = h.rank, cap = h.cap_s1;
    const int b0 = z * BT, nb = min(BT, h.batch - b0);
    const int parts = (r + kTile - 1) / kTile, ng = nw / parts;     // host: parts <= nw
    const int part = w % parts, g = w / parts, nq = d_in / 8;
    Channels<BT> ch{h.X, d_in, h.batch, b0, nb, 0, h.s1.wgs * nw, wg * nw + w, h.union_all != 0, {}};
    ch.n_ch = max(0, (nq - ch.first + ch.step - 1) / ch.step);
    uint32_t xr[kTokenPieces<BT>][BT];
    request_channels<BT>(ch, 0, xr);
    load_rules<BT, EXT>(L, b0, nb, ch.rules);
    if (!EXT) {
#pragma unroll
        for (int b = 0; b < BT; ++b) ch.rules.r[b].ge = h.tau_ge;
    }
    uint32_t *const s_off = reinterpret_cast<uint32_t *>(smem), *const s_cf = s_off + nw * cap;  // [nw * cap], [nw * cap][BT]
    float *const s_red = reinterpret_cast<float *>(s_cf + nw * cap * BT);                        // [nw][kTile]
    int *const s_misc = reinterpret_cast<int *>(s_red + (size_t)nw * kTile);
    const uint32_t pitch = (uint32_t)r * 2u;
    if (tid < 9) s_misc[tid] = tid == 0 ? 0 : 2 * ng * R;            // the list's length, the next batch of every part
    __syncthreads();
    compact_channels<DT, BT, EXT, true>(ch, L, pitch, xr, s_off, s_cf, s_misc, nullptr);
    __syncthreads();
    RS_STAMP(2);
    const int n = uniform(s_misc[0]), col = part * kTile + lane * 8;
    const SharedRows sr{s_off, s_cf, n, n, g * R, (ng + g) * R, s_misc + 1 + part, 0u, 0u};
    float acc[BT][8];
#pragma unroll
    for (int b = 0; b < BT; ++b)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[b][e] = 0.f;
    auto none = [](int, bool, unsigned long long (&)[BT]) {};
    // (waves past the last whole set of parts have none, and must not claim any either: what they claim nobody else streams)
    int done = 0;
    if (g < ng) done = stream_rows<DT, BT, NT, R>(buffer_of(h.SVc, (uint32_t)d_in * pitch), col < r ? (uint32_t)col * 2u : kOutside, sr, acc, none, none);
    RS_STAMP(3);
    RS_STAMP_SET(15, done);
    (void)done;
    // b must stay a compile-time index (a run-time subscript would push acc[][] into scratch memory)
    float *const t_sum = as_global(L.t_sum) + (size_t)z * BT * r;
#pragma unroll
    for (int b = 0; b < BT; ++b) {
        if (b >= nb) break;
        if (b > 0) __syncthreads();
        float4 *dst = reinterpret_cast<float4 *>(s_red + w * kTile + lane * 8);
        dst[0] = float4{acc[b][0], acc[b][1], acc[b][2], acc[b][3]};
        dst[1] = float4{acc[b][4], acc[b][5], acc[b][6], acc[b][7]};
        __syncthreads();
        for (int i = tid; i < parts * kTile; i += nthr) {
            const int pt = i / kTile, cl = i % kTile;
            float sum = 0.f;
            for (int gg = 0; gg < ng; ++gg) sum += s_red[(gg * parts + pt) * kTile + cl];
            if (i < r) __hip_atomic_fetch_add(t_sum + (size_t)b * r + i, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }

    // ---- arrive; the last stage-1 workgroup of the batch tile publishes its t
    int *const line = as_global(h.sync) + kSyncStage1 + z * kSyncLine;
    const uint32_t gen = generation(line);
    wait_own_writes();
    __syncthreads();
    RS_STAMP(4);
    if (tid == 0) s_misc[0] = __hip_atomic_fetch_add(line, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    RS_STAMP(5);
    if (s_misc[0] != h.s1.wgs - 1) {
        RS_STAMP_FLUSH(1, wg, w);
        return;
    }
    unsigned long long *const t_tag = as_global(h.t_tag);
    for (int i = tid; i < nb * r; i += nthr) {
        const float v = __hip_atomic_exchange(t_sum + i, 0.f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!h.s1.skip) publish_t(t_tag + (size_t)z * BT * r + i, gen, v);
    }
    RS_STAMP(6);
    RS_STAMP_FLUSH(3, wg, w);
    for (int i = tid; i < r; i += nthr) refresh_unused(t_tag, r, h.s1.t_slots, nb, z, gen, i);
    if (tid == 0) end_of_line(line);          // (every wave has used the generation: it came before the barriers)
}

template <int DT, int BT, bool NT, bool EXT, bool SVC, int R>
__device__ __forceinline__ void direct_body(const DirectGroupArgs &ga, unsigned char *smem)
{
    RS_STAMP_DECL;
    RS_STAMP(1);
    const int z = blockIdx.z;
    int wg;
    const int job = find_job(ga.wg_end, ga.n, blockIdx.x, wg);
    const DirectArgs &a = ga.job[job];
    const LayerView &L = a.L;
    DirectArgs h = a;
    __asm__ volatile("" : "+s"(h.X), "+s"(h.M), "+s"(h.sync), "+s"(h.t_tag), "+s"(h.yacc), "+s"(h.act_bits), "+s"(h.d_in), "+s"(h.d_out), "+s"(h.rank),
                     "+s"(h.batch), "+s"(h.tiles), "+s"(h.splits), "+s"(h.cap), "+s"(h.lr_wgs), "+s"(h.tiles_inv), "+s"(h.tile_map), "+s"(h.union_all),
                     "+s"(h.tau_ge), "+s"(h.q_base), "+s"(h.q_rem), "+s"(h.u_base), "+s"(h.u_rem), "+s"(h.waves), "+s"(h.SVc));
    RS_STAMP(2);
    const int lr_wgs = h.lr_wgs, n_tiles = h.tiles, n_splits = h.splits, d_in = h.d_in, d_out = h.d_out, cap = h.cap, rank = h.rank;
    if (__builtin_expect(wg < lr_wgs, 0)) {
        // every gather workgroup ends with rows that need t: the stage-1 waves issue ahead of the gather waves they
        // share a compute unit with (measured: q/k/v grouped at 8192 wide 37.0 -> 35.6 us, the other launches unchanged)
        __builtin_amdgcn_s_setprio(3);
        if constexpr (SVC) {
            if (h.SVc) {
                stage1_gather<DT, BT, NT, EXT, BT == 1 ? 8 : 4>(h, L, smem, wg, z);
                return;
            }
        }
        stage1_tagged<DT, BT, EXT>(a.s1, L, smem, wg, z);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, w = uniform(tid >> 6), nw = h.waves;
    int tile, split;
    if (h.tile_map != 2) {
        split = h.tiles_inv ? (int)__umulhi((uint32_t)(wg - lr_wgs), h.tiles_inv) : wg - lr_wgs;
        tile = wg - lr_wgs - split * n_tiles;
    } else if (!map_tile(2, n_tiles, n_splits, wg - lr_wgs, tile, split)) {
        return;
    }
    const int b0 = z * BT;
    const int nb = min(BT, h.batch - b0);
    const int rho = split * nw + w;
    Channels<BT> ch{h.X, d_in, h.batch, b0, nb, h.q_base + (rho < h.q_rem ? 1 : 0), n_splits * nw, rho, h.union_all != 0, {}};
    uint32_t xr[kTokenPieces<BT>][BT];
    request_channels<BT>(ch, 0, xr);
    int *const line = as_global(h.sync) + sync_tile(n_tiles, z, tile);
    const uint32_t gen = generation(line);
    load_rules<BT, EXT>(L, b0, nb, ch.rules);
    if (!EXT) {
#pragma unroll
        for (int b = 0; b < BT; ++b) ch.rules.r[b].ge = h.tau_ge;
    }
    uint32_t *const s_off = reinterpret_cast<uint32_t *>(smem), *const s_cf = s_off + nw * cap;  // [nw * cap], [nw * cap][BT]
    float *const s_red = reinterpret_cast<float *>(s_cf + nw * cap * BT);                        // [nw][kTile]
    int *const s_misc = reinterpret_cast<int *>(s_red + (size_t)nw * kTile);

    // ---- sigma_t on my channels, for the workgroup's list; the split's share of the rows of U_r^T follows as rows d_in + j of M
    //      with coefficients t
    const uint32_t pitch = (uint32_t)d_out * 2u;
    if (tid < 2) s_misc[tid] = tid == 0 ? 0 : 2 * nw * R;            // the list's length, the next batch
    __syncthreads();
    compact_channels<DT, BT, EXT, false>(ch, L, pitch, xr, s_off, s_cf, s_misc, tile == 0 ? as_global(h.act_bits) + (size_t)z * d_in : nullptr);
    __syncthreads();
    const int n = uniform(s_misc[0]), u_lo = split * h.u_base + min(split, h.u_rem), nu = h.u_base + (split < h.u_rem ? 1 : 0);
    const SharedRows sr{s_off, s_cf, n, n + nu, w * R, (nw + w) * R, s_misc + 1, (uint32_t)(d_in + u_lo) * pitch, pitch};
    RS_STAMP(3);

    // t of the rows behind the list: requested when their batch is, needed when the batch's turn comes
    const unsigned long long *const t_tag = as_global(h.t_tag) + (size_t)z * BT * rank + u_lo;
    auto request_t = [&](int j, bool has, unsigned long long (&q)[BT]) { request_tagged<BT>(t_tag, rank, nb, j, has, q); };
    auto settle_t = [&](int j, bool has, unsigned long long (&q)[BT]) {
        settle_tagged<BT>(t_tag, rank, nb, j, has, gen, a.wait_polls, as_global(h.sync), q);
        RS_STAMP(5);
    };
    float acc[BT][8];
#pragma unroll
    for (int b = 0; b < BT; ++b)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[b][e] = 0.f;
    const int col = tile * kTile + lane * 8;
    const int done = stream_rows<DT, BT, NT, R>(buffer_of(h.M, (uint32_t)(d_in + rank) * pitch), col < d_out ? (uint32_t)col * 2u : kOutside, sr, acc,
                                                request_t, settle_t);
    (void)done;
    RS_STAMP(6);
    RS_STAMP_SET(15, done);
    RS_STAMP_SET(14, ((unsigned)__builtin_amdgcn_s_getreg(20 | (3 << 11)) << 16) | ((unsigned)__builtin_amdgcn_s_getreg(4 | (31 << 11)) & 0xffff));
    reduce_to_yacc<BT>(acc, s_red, as_global(h.yacc), b0, nb, d_out, tile);
    RS_STAMP(7);

    // ---- arrive at the tile; the last of its `splits` workgroups owns the finish.  For a gate/up pair
    //      the two layers share the gate layer's counters and the tile is finished once, by the last
    //      of both layers' workgroups (Sec. 3.1: H = X W_up^T (.) silu(X W_gate^T)).
    wait_own_writes();
    __syncthreads();
    RS_STAMP(8);
    const bool pair = ga.gate_up != 0;
    int *const arrive = pair ? ga.job[0].L.sync + sync_tile(n_tiles, z, tile) : line;
    const int arrivals = pair ? ga.job[0].splits + ga.job[1].splits : n_splits;
    if (tid == 0) s_misc[0] = __hip_atomic_fetch_add(arrive, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    RS_STAMP(9);
    if (s_misc[0] != arrivals - 1) {
        RS_STAMP_FLUSH(0, wg, w);
        return;
    }

    finish_tile<DT, BT, EXT, kTile>(pair ? ga.job[0].L : L, pair ? &ga.job[1].L : nullptr, pair ? ga.job[0].L.yacc : as_global(h.yacc),
                                    pair ? ga.job[0].Y : a.Y, tile, b0, nb, d_out);
    RS_STAMP(10);
    RS_STAMP_FLUSH(2, wg, w);
    if (tid == 0) {
        end_of_line(arrive);
        if (pair) end_of_line(ga.job[1].L.sync + sync_tile(n_tiles, z, tile));
    }
}

// LDS carve-up of the gather part.
struct GatherLds {
    int *idx;
    float *coef;
    float *red;
    int *misc;
};
__device__ __forceinline__ GatherLds carve(unsigned char *smem, int cap, int bt, int nw)
{
    GatherLds s;
    s.red = reinterpret_cast<float *>(smem);                       // 16-byte aligned
    s.coef = s.red + (nw > 1 ? nw * kTile : 0);
    s.idx = reinterpret_cast<int *>(s.coef + (size_t)cap * bt);
    s.misc = s.idx + cap;
    return s;
}

// ---------------------------------------------------------------------------------------------
// 4-bit weights (Sec. 4.4: R-Sparse on GPTQ weights, groups of 128 input channels): W~[o][c] =
// s[o][g] (q[o][c] - z[o][g]).  A wave streams a CONTIGUOUS run of its workgroup's kept-channel list, so
// the channels of one quantisation group arrive together: it accumulates grp = sum_c x_c q_c and
// sumx = sum_c x_c while the group lasts and folds acc += s (grp - z sumx) once when it ends -- the
// codes go from nibble to float and into one FMA per token, nothing else per weight.  Scale and zero
// point of a group are requested when the group opens and used when it closes.
// A lane owns 16 output columns of a 1024-column tile: 8 bytes per row, words h = 0, 1 (layout: kernels.h).
// ---------------------------------------------------------------------------------------------
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// A batch of kUnroll rows as one register vector (word 2u + h = word h of row u): the rolled loop below
// picks a row by a run-time index, which the compiler serves with relative register addressing on a
// vector type (an array would go to scratch memory).
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
static_assert(kUnroll == 8, "u32x16 holds 8 rows of two words");

template <bool NT>
__device__ __forceinline__ u32x2 ldg8(const uint8_t *p)
{
    const u32x2 *q = reinterpret_cast<const u32x2 *>(p);
    return NT ? __builtin_nontemporal_load(q) : *q;
}

// kUnroll rows starting at list position j0 of a non-empty run that ends at j_hi.  Positions past the end
// re-read the run's last row (a cache hit) and are given a zero coefficient by the consumer, so that a batch
// is always eight unconditional loads: the compiler can then count outstanding loads exactly and lets the
// next batch stay in flight while this one is consumed.  Rows and the scale / zero-point rows are padded
// to whole tiles, so lanes past d_out read zeros instead of being masked off.
template <bool NT>
__device__ __forceinline__ void load_batch_q4(const uint8_t *__restrict__ Mq, size_t ld, int off, const int *s_idx,
                                              int j_hi, int j0, u32x16 &v)
{
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const int idx = uniform(s_idx[min(j0 + u, j_hi - 1)]);
        const u32x2 w = ldg8<NT>(Mq + (size_t)idx * ld + off);
        v[2 * u] = w[0];
        v[2 * u + 1] = w[1];
    }
}

// The eight codes of one word as floats: element e < 4 is the low nibble of byte e, element 4 + e its high nibble.
__device__ __forceinline__ void codes8(uint32_t w, float (&f)[8])
{
    uint32_t lo = w & 0x0f0f0f0fu, hi = (w >> 4) & 0x0f0f0f0fu;
    // keep the two masked words as they are: each byte then converts with one byte-select instruction,
    // where the compiler would otherwise extract every nibble with a bit-field op first
    __asm__ volatile("" : "+v"(lo), "+v"(hi));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f[k] = (float)((lo >> (8 * k)) & 0xffu);
        f[4 + k] = (float)((hi >> (8 * k)) & 0xffu);
    }
}

template <int BT>
struct Q4State {
    float acc[2][BT][8];    // finished groups, scaled
    float grp[2][BT][8];    // sum_c x_c q_c of the open group
    float sumx[BT];         // sum_c x_c of the open group
    u32x4 sv[2];            // scales of the open group, 8 columns per word h
    u32x2 zv[2];            // its zero points, one byte per column
    int g;                  // the open group, -1 = none
};

template <int BT>
__device__ __forceinline__ void q4_open(Q4State<BT> &st, const LayerView &L, int g, int colq)
{
    st.g = g;
    const size_t at = (size_t)g * ((size_t)L.qtiles * kQ4Tile) + colq;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        st.sv[h] = *reinterpret_cast<const u32x4 *>(L.qs + at + h * 512);
        st.zv[h] = *reinterpret_cast<const u32x2 *>(L.qz + at + h * 512);
    }
}

template <int DT, int BT>
__device__ __forceinline__ void q4_close(Q4State<BT> &st)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        float sf[8];
        unpack8<DT>(st.sv[h], sf);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t zw = st.zv[h][e >> 2];
            const float zf = (float)((zw >> (8 * (e & 3))) & 0xffu);
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                const float d = __builtin_fmaf(-zf, st.sumx[b], st.grp[h][b][e]);
                st.acc[h][b][e] = __builtin_fmaf(sf[e], d, st.acc[h][b][e]);
                st.grp[h][b][e] = 0.f;
            }
        }
    }
#pragma unroll
    for (int b = 0; b < BT; ++b) st.sumx[b] = 0.f;
}

// One row: its 16 codes times the token coefficients, into the open group's sums.
template <int BT>
__device__ __forceinline__ void q4_row(Q4State<BT> &st, const u32x2 w, const float *s_coef, int j, int j_hi)
{
    float cf[BT];
#pragma unroll
    for (int b = 0; b < BT; ++b) {
        cf[b] = uniform(s_coef[min(j, j_hi - 1) * BT + b]);
        cf[b] = j < j_hi ? cf[b] : 0.f;
        st.sumx[b] += cf[b];
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        float f[8];
        codes8(w[h], f);
#pragma unroll
        for (int b = 0; b < BT; ++b)
#pragma unroll
            for (int e = 0; e < 8; ++e) st.grp[h][b][e] = __builtin_fmaf(cf[b], f[e], st.grp[h][b][e]);
    }
}

// A batch of up to kUnroll rows.  The list is ascending, so when its first and last row lie in the open
// group all of them do: that common case is straight-line code.  A batch that crosses a group boundary
// takes the rolled loop, which holds the only copy of the fold (close) and of the scale request (open).
template <int DT, int BT>
__device__ __forceinline__ void q4_consume(Q4State<BT> &st, const LayerView &L, const u32x16 &v,
                                           const int *s_idx, const float *s_coef, int j_hi, int j0, int colq)
{
    const int j_last = min(j0 + kUnroll, j_hi) - 1;
    const int g_first = uniform(s_idx[j0]) >> L.qshift, g_last = uniform(s_idx[j_last]) >> L.qshift;
    if (g_first == st.g && g_last == st.g) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) q4_row<BT>(st, u32x2{v[2 * u], v[2 * u + 1]}, s_coef, j0 + u, j_hi);
    } else {
#pragma unroll 1
        for (int u = 0; u < kUnroll; ++u) {
            if (j0 + u >= j_hi) break;
            const int g = uniform(s_idx[j0 + u]) >> L.qshift;
            if (g != st.g) {
                if (st.g >= 0) q4_close<DT, BT>(st);
                q4_open<BT>(st, L, g, colq);
            }
            q4_row<BT>(st, u32x2{v[2 * u], v[2 * u + 1]}, s_coef, j0 + u, j_hi);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// First launch of the layer.  Workgroups [0, lr_wgs) compute stage 1 of the low-rank part; the
// others do steps 1-2 of the sparse part: sparsification mask and ascending kept-channel list
// (Sec. 3.4, sigma_t) -- every workgroup scans the whole token and keeps its balanced share --
// then the gather-GEMV over the kept columns of W, accumulated into yacc with fp32 atomics.
// The two groups are independent, so they share one launch.
// grid.x = lr_wgs + tiles * splits, grid.z = batch tiles of BT tokens, block = 64 * waves.
// ---------------------------------------------------------------------------------------------
template <int DT, int BT, bool NT, bool Q4>
__device__ __forceinline__ void sparse_body(const GroupArgs &ga, unsigned char *smem)
{
    constexpr int R = kUnroll;
    const int z = blockIdx.z;
    int wg;
    const GatherArgs &a = ga.job[find_job(ga.wg_end, ga.n, blockIdx.x, wg)];
    const LayerView &L = a.L;
    // everything the path to the first weight load needs, fetched in one go
    const int lr_wgs = pin(a.lr_wgs), tile_map = pin(a.tile_map), n_tiles = pin(a.tiles), n_splits = pin(a.splits);
    const uint16_t *const X = pin(a.X);
    const int d_in = pin(L.d_in), d_out = pin(L.d_out), batch = pin(a.batch), cap = pin(a.cap);
    const bool union_all = pin(L.batch_mask_mode) == 1;
    if (__builtin_expect(wg < lr_wgs, 0)) {
        lowrank_rows<DT, BT, kPubPlain>(RowsArgs{a.X, a.batch, a.lr_rows, a.lr_chunk, 0, lr_wgs, 0}, L, smem, wg, z);
        return;
    }
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, w = tid >> 6, nw = nthr >> 6;
    int tile, split;
    if (!map_tile(tile_map, n_tiles, n_splits, wg - lr_wgs, tile, split)) return;
    const int b0 = z * BT;
    const int nb = min(BT, batch - b0);
    TileRules<BT> rules;
    load_rules<BT, true>(L, b0, nb, rules);
    const GatherLds s = carve(smem, cap, BT, nw);
    const int col = tile * kTile + lane * 8;
    const bool colok = col < d_out;

    // ---- pass 1, coalesced over the token(s): keep-bits of every 8 channels (union over the batch
    //      tile, or over the whole batch with the union mask).  A wave covers 64 consecutive 8-channel
    //      chunks at a time and scans their kept counts in registers straight away; per chunk it leaves
    //      the keep-bits and the count of kept channels before it inside those 64 chunks, per 64 chunks
    //      their total.  No barrier up to here: every thread only touches its own slots.
    const int nq = d_in / 8;
    uint8_t *s_u = reinterpret_cast<uint8_t *>(s.misc + 16);
    int *s_P = reinterpret_cast<int *>(s_u + ((nq + 3) & ~3));
    const int E = (nq + 63) >> 6;                      // blocks of 64 chunks
    int *s_tot = s_P + nq, *s_base = s_tot + E;
    constexpr int PB = TokenBatch<BT>::kGroups;
    // every list slot starts as a valid channel, so that no later arithmetic slip can turn LDS leftovers into addresses
    for (int i = tid; i < cap; i += nthr) s.idx[i] = 0;
    for (int qb = w * 64; qb < nq; qb += nthr * PB) {
        u32x4 raw[PB][BT];
#pragma unroll
        for (int p = 0; p < PB; ++p)
            if (qb + p * nthr + lane < nq) load_raw8<BT>(X, b0, nb, d_in, (qb + p * nthr + lane) * 8, raw[p]);
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int qrow = qb + p * nthr;            // first chunk of this wave's block: the same for all its lanes
            if (qrow < nq) {
                const int q = qrow + lane;
                uint32_t kept = 0u;
                if (q < nq) {
                    uint32_t m[BT];
                    kept = masks_of8<DT, BT>(L, X, batch, b0, nb, d_in, q * 8, rules, union_all, raw[p], m);
                    if (Q4 && a.dense) kept = 0xffu;
                }
                const int c = __popc(kept);
                const int inc = wave_inclusive_scan(c);
                if (q < nq) {
                    s_u[q] = (uint8_t)kept;
                    s_P[q] = inc - c;
                }
                if (lane == 63) s_tot[qrow >> 6] = inc;
            }
        }
    }
    __syncthreads();

    // ---- pass 2: every wave turns the block totals into block bases for itself (identical values from
    //      every wave, read back only by the wave that wrote them), which also gives the list length k
    int k = 0;
    for (int eb = 0; eb < E; eb += 64) {
        const int e = eb + lane;
        const int v = e < E ? s_tot[e] : 0;
        const int inc = wave_inclusive_scan(v);
        if (e < E) s_base[e] = k + inc - v;
        k += __shfl(inc, 63, 64);
    }
    k = min(max(uniform(k), 0), d_in);

    // ---- my balanced share [lo, hi) of the ascending kept list: each thread writes out the entries of its
    //      own chunks that fall into it
    int lo, hi;
    balanced_share(k, n_splits, split, lo, hi);
    const int n = hi - lo;
    for (int qrow = w * 64; qrow < nq; qrow += nthr) {
        const int q = qrow + lane;
        if (q < nq) {
            const uint32_t u = s_u[q];
            const int P = s_base[qrow >> 6] + s_P[q];
            if (u != 0u && P < hi && P + __popc(u) > lo) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int p = P + __popc(u & ((1u << e) - 1u));
                    if (((u >> e) & 1u) && p >= lo && p < hi) s.idx[p - lo] = q * 8 + e;
                }
            }
        }
    }
    if (tile == 0 && split == 0 && tid == 0) L.act_count[z] = k;
    __syncthreads();

    // ---- issue the first batch of weight loads (they need only the indices) ...
    float acc[BT][8];
#pragma unroll
    for (int b = 0; b < BT; ++b)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[b][e] = 0.f;
    u32x4 va[R];
    const int j_first = w * R, step = nw * R;
    // 4-bit weights: this wave's contiguous run [jq_lo, jq_hi) of the list, 8 bytes per lane and row
    // (wave index and row count go through readfirstlane: the compiler cannot know they are wave-uniform, and
    //  would otherwise run the row loop and the group tests under execution masks)
    const int wq = uniform(w), nq_rows = uniform(n);
    int jq_lo, jq_hi;
    balanced_share(nq_rows, nw, wq, jq_lo, jq_hi);
    const int colq = tile * kQ4Tile + lane * 8;
    const size_t ldq = (size_t)L.qtiles * (kQ4Tile / 2);
    const int offq = tile * (kQ4Tile / 2) + lane * 8;
    u32x16 qa, qb;
    Q4State<Q4 ? BT : 1> st;
    if constexpr (Q4) {
        st.g = -1;
        if (jq_lo < jq_hi) {
            // two batches of rows and the first group's scale and zero point are requested before the
            // coefficients are fetched: a wave with up to 16 rows has everything in flight at once
            load_batch_q4<NT>(L.Mq, ldq, offq, s.idx, jq_hi, jq_lo, qa);
            load_batch_q4<NT>(L.Mq, ldq, offq, s.idx, jq_hi, jq_lo + kUnroll, qb);
            q4_open<BT>(st, L, uniform(s.idx[jq_lo]) >> L.qshift, colq);
        }
    } else {
        load_batch<NT, R>(L.M, (size_t)d_out, col, colok, s.idx, n, j_first, va);
    }

    // ---- ... and fetch the coefficients x[b, c] * m[b, c] of my rows while those loads fly
    for (int j = tid; j < n; j += nthr) {
        const int c = s.idx[j];
        uint32_t bits = 0;
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            float xf = 0.f;
            bool kb = false;
            if (b < nb) {
                const uint16_t h = X[(size_t)(b0 + b) * d_in + c];
                xf = (DT == F16) ? (float)__builtin_bit_cast(_Float16, h) : as_f((uint32_t)h << 16);
                kb = (union_all || (Q4 && a.dense)) ? true
                     : rules.exact ? keep(xf, c, rules.r[b], rules.sgn) : keep_threshold(xf, rules.r[b]);
            }
            s.coef[j * BT + b] = kb ? xf : 0.f;
            bits |= (uint32_t)kb << b;
        }
        if (tile == 0) {          // the tile-0 workgroups publish the list for read-back
            L.act_list[(size_t)z * d_in + lo + j] = c;
            L.act_bits[(size_t)z * d_in + lo + j] = bits;
        }
    }
    __syncthreads();

    if constexpr (Q4) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int b = 0; b < BT; ++b)
#pragma unroll
                for (int e = 0; e < 8; ++e) { st.acc[h][b][e] = 0.f; st.grp[h][b][e] = 0.f; }
#pragma unroll
        for (int b = 0; b < BT; ++b) st.sumx[b] = 0.f;
        for (int j0 = jq_lo; j0 < jq_hi; j0 += 2 * kUnroll) {
            q4_consume<DT, BT>(st, L, qa, s.idx, s.coef, jq_hi, j0, colq);
            if (j0 + kUnroll >= jq_hi) break;
            load_batch_q4<NT>(L.Mq, ldq, offq, s.idx, jq_hi, j0 + 2 * kUnroll, qa);
            q4_consume<DT, BT>(st, L, qb, s.idx, s.coef, jq_hi, j0 + kUnroll, colq);
            if (j0 + 2 * kUnroll >= jq_hi) break;
            load_batch_q4<NT>(L.Mq, ldq, offq, s.idx, jq_hi, j0 + 3 * kUnroll, qb);
        }
        if (st.g >= 0) q4_close<DT, BT>(st);
        // the two 512-column halves of the tile go through the 16-bit path's reduction one after the other
        reduce_to_yacc<BT>(st.acc[0], s.red, L.yacc, b0, nb, d_out, tile * 2);
        __syncthreads();
        reduce_to_yacc<BT>(st.acc[1], s.red, L.yacc, b0, nb, d_out, tile * 2 + 1);
    } else {
        stream_rest<DT, BT, NT, R>(L.M, (size_t)d_out, col, colok, s.idx, s.coef, n, j_first, step, va, acc, [](int) {});
        reduce_to_yacc<BT>(acc, s.red, L.yacc, b0, nb, d_out, tile);
    }
}

// 4-bit weights, up to 4 tokens: the same scan, list and stage-1 workgroups, the weight stream as above.
// (four tokens need two sets of 16 x 4 accumulators: at most 4 waves per workgroup, one per SIMD, so that a
//  wave may use the whole register file)
template <int DT, int BT, bool NT>
__global__ __launch_bounds__(BT >= 4 ? 256 : 512) void k_q4_sparse_and_t(const GroupArgs ga)
{
    extern __shared__ __align__(16) unsigned char smem[];
    sparse_body<DT, BT, NT, true>(ga, smem);
}

// Eight tokens of accumulators need the full register file: 4 waves per workgroup, one per SIMD.
template <int DT, int BT, bool NT>
__global__ __launch_bounds__(BT >= 8 ? 256 : 512) void k_sparse_and_t(const GroupArgs ga)
{
    extern __shared__ __align__(16) unsigned char smem[];
    sparse_body<DT, BT, NT, false>(ga, smem);
}

// The whole layer in one launch (see the file header).  Same grid as k_sparse_and_t.
// EXT = false: no layer of the launch has a fixed-count rule, a signed threshold or a bias (the host checks), and the
// code for those is left out -- this kernel's once-per-launch code runs from a cold instruction cache.
// SVC: some layer of the launch takes stage 1 over its channel-major copy.
// R: rows per batch of loads of a wave: four (two batches of 4 KiB in flight; with eight 0 to 3 % slower).
template <int DT, int BT, bool NT, bool EXT, bool SVC, int R>
__global__ __launch_bounds__(BT >= 8 ? 256 : 512, BT >= 8 ? 3 : 4) void k_rsparse_fused(const DirectGroupArgs ga)
{
    extern __shared__ __align__(16) unsigned char smem[];
    direct_body<DT, BT, NT, EXT, SVC, R>(ga, smem);
}

// ---------------------------------------------------------------------------------------------
// Dense baseline, axpy form over the same column-major W: every channel, no mask, no low rank.
// Followed by k_finish with rank 0.
// ---------------------------------------------------------------------------------------------
template <int DT, int BT, bool NT>
__global__ __launch_bounds__(BT >= 8 ? 256 : 512) void k_dense_axpy(const GroupArgs ga)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, w = tid >> 6, nw = nthr >> 6;
    const int z = blockIdx.z;
    int wg;
    const GatherArgs &a = ga.job[find_job(ga.wg_end, ga.n, blockIdx.x, wg)];
    int tile, split;
    if (!map_tile(a, wg, tile, split)) return;
    const LayerView &L = a.L;
    const int d_in = L.d_in, d_out = L.d_out;
    const int b0 = z * BT;
    const int nb = min(BT, a.batch - b0);
    const GatherLds s = carve(smem, a.cap, BT, nw);

    int lo, hi;
    balanced_share(d_in, a.splits, split, lo, hi);
    const int n = hi - lo;
    for (int j = tid; j < n; j += nthr) {
        s.idx[j] = lo + j;
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            float xf = 0.f;
            if (b < nb) {
                const uint16_t h = a.X[(size_t)(b0 + b) * d_in + lo + j];
                xf = (DT == F16) ? (float)__builtin_bit_cast(_Float16, h) : as_f((uint32_t)h << 16);
            }
            s.coef[j * BT + b] = xf;
        }
    }
    __syncthreads();

    const int col = tile * kTile + lane * 8;
    const bool colok = col < d_out;
    float acc[BT][8];
#pragma unroll
    for (int b = 0; b < BT; ++b)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[b][e] = 0.f;
    u32x4 va[kUnroll];
    load_batch<NT, kUnroll>(L.M, (size_t)d_out, col, colok, s.idx, n, w * kUnroll, va);
    stream_rest<DT, BT, NT, kUnroll>(L.M, (size_t)d_out, col, colok, s.idx, s.coef, n, w * kUnroll, nw * kUnroll, va, acc,
                            [](int) {});
    reduce_to_yacc<BT>(acc, s.red, L.yacc, b0, nb, d_out, tile);
}

// ---------------------------------------------------------------------------------------------
// Second launch: steps 3b-4 of the layer.  Y[b, o] = round(yacc[b, o] + U_r[o, :] . t[b, :]), a row
// dot over U_r [d_out][rank] row-major (no cross-workgroup reduction), then yacc is re-zeroed for
// the next call.  LPR = lanes that cover one row of U_r (power of two, 16 bytes per lane and pass);
// a wave handles 64/LPR rows per pass.  rank == 0 just rounds yacc.
// grid.x workgroups of 4 waves over row groups, grid.z batch tiles.
// ---------------------------------------------------------------------------------------------
struct FinishArgs {
    LayerView L;
    void *Y;
    int batch, lpr, passes, use_rank;
};

constexpr int kFinishGroups = 4;     // row groups per wave, all loads issued up front
struct FinishGroupArgs {
    FinishArgs job[kMaxGroup];
    int wg_end[kMaxGroup];
    int n;
};

// PASSES = 16-byte pieces per lane and row (rank <= 512 * PASSES); 0 = any rank, loads not batched.
template <int DT, int BT, int PASSES>
__global__ __launch_bounds__(256) void k_finish(const FinishGroupArgs ga)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int z = blockIdx.z;
    int wg;
    const FinishArgs &a = ga.job[find_job(ga.wg_end, ga.n, blockIdx.x, wg)];
    const LayerView &L = a.L;
    const int d_out = L.d_out, r = a.use_rank;
    const int b0 = z * BT;
    const int nb = min(BT, a.batch - b0);
    float *s_t = reinterpret_cast<float *>(smem);             // [BT][r]
    const int lpr = a.lpr, rpi = 64 / lpr;                    // lanes per row, rows per wave and group
    const int sub = lane % lpr, rsel = lane / lpr;
    const int o_wave = (wg * 4 + w) * (rpi * kFinishGroups);
    constexpr int NP = PASSES > 0 ? PASSES : 1;

    // U_r rows and the accumulators first: their latency covers the staging of t
    u32x4 v[kFinishGroups][NP];
    float ya[kFinishGroups][BT];
#pragma unroll
    for (int g = 0; g < kFinishGroups; ++g) {
        const int o = o_wave + g * rpi + rsel;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int i = (p * lpr + sub) * 8;
            v[g][p] = (PASSES > 0 && o < d_out && i < r) ? ldg16<true>(L.U + (size_t)o * r + i) : u32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int b = 0; b < BT; ++b)
            ya[g][b] = (sub == 0 && o < d_out && b < nb) ? L.yacc[(size_t)(b0 + b) * d_out + o] : 0.f;
    }
    {   // stage t [BT][r] in LDS: four values per thread and step, eight steps of loads in flight
        constexpr int SB = 8;
        const int total4 = BT * r / 4;                     // r is a multiple of 8
        const float4 *src = reinterpret_cast<const float4 *>(L.t + ((size_t)z * BT) * r);
        for (int i0 = tid; i0 < total4; i0 += 256 * SB) {
            float4 tv[SB];
#pragma unroll
            for (int u = 0; u < SB; ++u) {
                const int i = i0 + u * 256;
                tv[u] = (i < total4 && (i * 4) / r < nb) ? src[i] : float4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int u = 0; u < SB; ++u) {
                const int i = i0 + u * 256;
                if (i < total4) reinterpret_cast<float4 *>(s_t)[i] = tv[u];
            }
        }
    }
    __syncthreads();

    float acc[kFinishGroups][BT];
#pragma unroll
    for (int g = 0; g < kFinishGroups; ++g) {
        const int o = o_wave + g * rpi + rsel;
#pragma unroll
        for (int b = 0; b < BT; ++b) acc[g][b] = 0.f;
        if (PASSES > 0) {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int i = (p * lpr + sub) * 8;
                if (o < d_out && i < r) {
                    float f[8];
                    unpack8<DT>(v[g][p], f);
#pragma unroll
                    for (int b = 0; b < BT; ++b) {
                        const float4 t0 = *reinterpret_cast<const float4 *>(s_t + b * r + i);
                        const float4 t1 = *reinterpret_cast<const float4 *>(s_t + b * r + i + 4);
                        float s = acc[g][b];
                        s = __builtin_fmaf(f[0], t0.x, s); s = __builtin_fmaf(f[1], t0.y, s);
                        s = __builtin_fmaf(f[2], t0.z, s); s = __builtin_fmaf(f[3], t0.w, s);
                        s = __builtin_fmaf(f[4], t1.x, s); s = __builtin_fmaf(f[5], t1.y, s);
                        s = __builtin_fmaf(f[6], t1.z, s); s = __builtin_fmaf(f[7], t1.w, s);
                        acc[g][b] = s;
                    }
                }
            }
        } else if (o < d_out) {
            for (int p = 0; p < a.passes; ++p) {
                const int i = (p * lpr + sub) * 8;
                if (i < r) {
                    float f[8];
                    unpack8<DT>(ldg16<true>(L.U + (size_t)o * r + i), f);
#pragma unroll
                    for (int b = 0; b < BT; ++b)
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc[g][b] = __builtin_fmaf(f[e], s_t[b * r + i + e], acc[g][b]);
                }
            }
        }
    }
    // Segmented butterfly over the lpr lanes of a row.  The distance is a compile-time constant and
    // all groups x tokens move together, so the cross-lane operations of one step overlap instead of
    // each waiting for the previous one.
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        if (d < lpr) {
#pragma unroll
            for (int g = 0; g < kFinishGroups; ++g)
#pragma unroll
                for (int b = 0; b < BT; ++b) acc[g][b] += __shfl_xor(acc[g][b], d, 64);
        }
    }
#pragma unroll
    for (int g = 0; g < kFinishGroups; ++g) {
        const int o = o_wave + g * rpi + rsel;
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            if (sub == 0 && o < d_out && b < nb) {
                store_out(a.Y, (size_t)(b0 + b) * d_out + o, ya[g][b] + acc[g][b] + bias_at(L, o), L.out_dtype);
                L.yacc[(size_t)(b0 + b) * d_out + o] = 0.f;
            }
        }
    }
}

int batch_tile(int batch)
{
    if (batch <= 1) return 1;
    if (batch <= 2) return 2;
    if (batch <= 4) return 4;
    return 8;
}

int gather_cap(int d_in, int splits) { return (d_in + splits - 1) / splits + 2; }

// List slots of a wave of the one-launch kernel: all channels of its chunks.
int direct_cap(int d_in, int R) { return (d_in / 8 + R - 1) / R * 8; }
size_t direct_lds(int cap, int waves, int bt) { return (size_t)waves * (cap * (1 + bt) + kTile) * 4 + 64; }

int lowrank_chunk(int d_in, int bt)
{
    int chunk = (24576 / bt) & ~7;
    return d_in < chunk ? d_in : chunk;
}

}  // namespace

size_t gather_lds_bytes(int d_in, int splits, int waves, int bt)
{
    const size_t cap = gather_cap(d_in, splits);
    return (waves > 1 ? (size_t)waves * kTile * 4 : 0) + cap * bt * 4 + cap * 4 + 16 * 4 + (size_t)d_in / 8 + 16 +
           (size_t)d_in / 2 + 4 + 2 * ((size_t)d_in / 512 + 2) * 4;   // ... + keep-bits of every 8 channels + their list positions
}

size_t direct_lds_bytes(int d_in, int splits, int waves, int bt) { return direct_lds(direct_cap(d_in, splits * waves), waves, bt); }

bool direct_supported(int d_in, int d_out, int rank) { return (unsigned long long)(d_in + rank) * (unsigned)d_out * 2u <= kMaxBufferBytes; }

bool lowrank_copy_supported(int d_in, int rank) { return (unsigned long long)d_in * rank * 2u <= kMaxBufferBytes; }

size_t lowrank_lds_bytes(int d_in, int bt)
{
    return (size_t)bt * lowrank_chunk(d_in, bt) * 2 + 16;
}

// Unstaged, every set of two rows (four up to two tokens) reads and masks the tokens again: where a workgroup of four tokens has more
// rows than `unstaged`, and always at eight tokens, they are masked once, in LDS (us per call at 4, 8 and 16 rows a workgroup, unstaged -
// staged, four tokens, fixed count, 4096 x 4096, rank 256 22.8 - 22.7, 28.7 - 22.7, 40.0 - 24.3; 8192 x 8192, rank 512 40.6 - 42.9,
// 43.3 - 43.3, 65.2 - 43.6; 28672 -> 8192, rank 1024 8 rows 92.0 - 97.1; eight tokens, default rows: q/k/v of 8192 / 1024, rank
// 1024 342 - 90, gate and up of 4096 / 11008, rank 512 120 - 76).  The one-launch kernel of columns masks anew up to eight rows in
// launches of 2^25 weights or more, which hide it, and up to four in smaller ones (gate / up of 2048 / 5632, rank 256, five
// rows, fixed count: 32.0 - 27.9).  The strip kernel, one workgroup per compute unit at four
// tokens, gains from five rows on (8 rows: 4096 x 4096 20.2 - 16.6, 28672 -> 8192 125 - 107; 4 rows: 16.3 - 16.5, 118 - 116).
int stage1_chunk(int d_in, int bt, int rows, int unstaged)
{
    return bt >= 8 || (bt == 4 && rows > unstaged) ? lowrank_chunk(d_in, bt) : 0;
}

size_t stage1_lds_bytes(int d_in, int bt, int chunk)
{
    return chunk > 0 ? lowrank_lds_bytes(d_in, bt) : (size_t)2 * 8 * 8 * 4;     // stage1_rows: two sums of the waves
}

#define RS_DISPATCH_BT(BTV, ...)                      \
    switch (BTV) {                                    \
    case 1: { constexpr int BT = 1; __VA_ARGS__; } break; \
    case 2: { constexpr int BT = 2; __VA_ARGS__; } break; \
    case 4: { constexpr int BT = 4; __VA_ARGS__; } break; \
    default: { constexpr int BT = 8; __VA_ARGS__; } break; \
    }

static bool same_shape_class(const LayerView *L, int n)
{
    for (int i = 1; i < n; ++i)
        if (L[i].d_in != L[0].d_in || L[i].dtype != L[0].dtype) return false;
    return n >= 1 && n <= kMaxGroup;
}

hipError_t launch_sparse_and_t(const LayerView *L, const Launch *cfg, int n, const void *X, int batch, bool with_t,
                               bool with_gather, hipStream_t stream)
{
    if (!same_shape_class(L, n)) return hipErrorInvalidValue;
    const int bt = batch_tile(batch);
    const int nz = (batch + bt - 1) / bt;
    GroupArgs ga{};
    ga.n = n;
    size_t lds = 0;
    int total = 0;
    for (int i = 0; i < n; ++i) {
        GatherArgs &a = ga.job[i];
        const int tiles = (L[i].d_out + kTile - 1) / kTile;
        a.L = L[i]; a.X = (const uint16_t *)X; a.batch = batch; a.splits = cfg[i].splits; a.tiles = tiles;
        a.cap = gather_cap(L[i].d_in, cfg[i].splits);
        a.lr_wgs = (with_t && L[i].rank > 0) ? (L[i].rank + cfg[i].lowrank_rows - 1) / cfg[i].lowrank_rows : 0;
        a.lr_rows = cfg[i].lowrank_rows;
        a.lr_chunk = lowrank_chunk(L[i].d_in, bt);
        a.tile_map = cfg[i].tile_map;
        const int gather_wgs = !with_gather ? 0
                               : cfg[i].tile_map == 2 ? ((tiles + 7) / 8) * 8 * cfg[i].splits : tiles * cfg[i].splits;
        total += a.lr_wgs + gather_wgs;
        ga.wg_end[i] = total;
        lds = std::max(lds, gather_lds_bytes(L[i].d_in, cfg[i].splits, cfg[0].waves, bt));
        if (a.lr_wgs > 0) lds = std::max(lds, lowrank_lds_bytes(L[i].d_in, bt));
    }
    for (int i = n; i < kMaxGroup; ++i) ga.wg_end[i] = total;
    if (total == 0) return hipSuccess;
    if (lds > 64 * 1024) return hipErrorInvalidValue;
    dim3 grid(total, 1, nz), block(kWave * cfg[0].waves);
    const bool nt = cfg[0].nontemporal != 0;
#define RS_G(DT)                                                                                       \
    RS_DISPATCH_BT(bt, {                                                                               \
        if (nt) hipLaunchKernelGGL((k_sparse_and_t<DT, BT, true>), grid, block, lds, stream, ga);      \
        else hipLaunchKernelGGL((k_sparse_and_t<DT, BT, false>), grid, block, lds, stream, ga);        \
    })
    if (L[0].dtype == F16) { RS_G(F16) } else { RS_G(BF16) }
#undef RS_G
    return hipGetLastError();
}

hipError_t launch_q4(const LayerView *L, const Launch *cfg, int n, const void *X, int batch, bool with_t, bool dense, hipStream_t stream)
{
    if (!same_shape_class(L, n) || batch < 1 || batch > 32) return hipErrorInvalidValue;
    // batches above 4 tokens run as batch tiles of 4 in the grid's z dimension (the codes are streamed once per tile)
    const int bt = std::min(4, batch_tile(batch));
    const int nz = (batch + bt - 1) / bt;
    if (bt >= 4 && cfg[0].waves > 4) return hipErrorInvalidValue;
    GroupArgs ga{};
    ga.n = n;
    int total = 0;
    size_t lds = 0;
    for (int i = 0; i < n; ++i) {
        const LayerView &l = L[i];
        if (!l.Mq || !l.qs || !l.qz || l.qshift < 3 || (l.d_in >> l.qshift) < 1 || ((l.d_in >> l.qshift) << l.qshift) != l.d_in ||
            l.qtiles != (l.d_out + kQ4Tile - 1) / kQ4Tile || cfg[i].splits < 1 || cfg[i].lowrank_rows < 1 || cfg[i].lowrank_rows > kRowsPerWave * cfg[0].waves)
            return hipErrorInvalidValue;
        GatherArgs &a = ga.job[i];
        a.L = l; a.X = (const uint16_t *)X; a.batch = batch; a.splits = cfg[i].splits; a.tiles = l.qtiles;
        a.cap = gather_cap(l.d_in, cfg[i].splits);
        a.lr_wgs = (with_t && !dense && l.rank > 0) ? (l.rank + cfg[i].lowrank_rows - 1) / cfg[i].lowrank_rows : 0;
        a.lr_rows = cfg[i].lowrank_rows;
        a.lr_chunk = lowrank_chunk(l.d_in, bt);
        a.tile_map = 1;
        a.dense = dense ? 1 : 0;
        total += a.lr_wgs + l.qtiles * cfg[i].splits;
        ga.wg_end[i] = total;
        lds = std::max(lds, gather_lds_bytes(l.d_in, cfg[i].splits, cfg[0].waves, bt));
        if (a.lr_wgs > 0) lds = std::max(lds, lowrank_lds_bytes(l.d_in, bt));
    }
    for (int i = n; i < kMaxGroup; ++i) ga.wg_end[i] = total;
    if (lds > 64 * 1024) return hipErrorInvalidValue;
    dim3 grid(total, 1, nz), block(kWave * cfg[0].waves);
    const bool nt = cfg[0].nontemporal != 0;
#define RS_Q1(DT, BTV)                                                                                  \
    do {                                                                                                \
        if (nt) hipLaunchKernelGGL((k_q4_sparse_and_t<DT, BTV, true>), grid, block, lds, stream, ga);   \
        else hipLaunchKernelGGL((k_q4_sparse_and_t<DT, BTV, false>), grid, block, lds, stream, ga);     \
    } while (0)
#define RS_Q(DT)                     \
    switch (bt) {                    \
    case 1: RS_Q1(DT, 1); break;     \
    case 2: RS_Q1(DT, 2); break;     \
    default: RS_Q1(DT, 4); break;    \
    }
    if (L[0].dtype == F16) { RS_Q(F16) } else { RS_Q(BF16) }
#undef RS_Q1
#undef RS_Q
    return hipGetLastError();
}

hipError_t launch_fused(const LayerView *L, const Launch *cfg, int n, const void *X, int batch, void *const *Y,
                        hipStream_t stream, bool gate_up)
{
    if (!same_shape_class(L, n)) return hipErrorInvalidValue;
    if (gate_up && (n != 2 || L[0].d_out != L[1].d_out || L[0].out_dtype != L[0].dtype || cfg[0].tile_map == 2 ||
                    cfg[1].tile_map == 2))
        return hipErrorInvalidValue;
    const int bt = batch_tile(batch);
    const int nz = (batch + bt - 1) / bt;
    if (nz > kSyncMaxZ) return hipErrorInvalidValue;
    DirectGroupArgs ga{};
    ga.n = n;
    size_t lds = 0, weights = 0;
    for (int i = 0; i < n; ++i) weights += (size_t)L[i].d_in * L[i].d_out;
    int total = 0;
    for (int i = 0; i < n; ++i) {
        if (!L[i].sync || !Y[i]) return hipErrorInvalidValue;
        DirectArgs &h = ga.job[i];
        const int tiles = (L[i].d_out + kTile - 1) / kTile;
        if (!L[i].M || cfg[i].splits < 1 || !direct_supported(L[i].d_in, L[i].d_out, L[i].rank) || (L[i].rank > 0 && (!L[i].t_tag || L[i].t_slots < nz * bt)))
            return hipErrorInvalidValue;
        const int R_all = cfg[i].splits * cfg[0].waves;
        h.lr_wgs = L[i].rank > 0 ? (L[i].rank + cfg[i].lowrank_rows - 1) / cfg[i].lowrank_rows : 0;
        if (h.lr_wgs > 0 && (cfg[i].lowrank_rows < 1 || (bt >= 4 && cfg[i].lowrank_rows > kRowsPerWave * cfg[0].waves))) return hipErrorInvalidValue;
        const int chunk = stage1_chunk(L[i].d_in, bt, cfg[i].lowrank_rows, weights >= ((size_t)1 << 25) ? 8 : 4);
        size_t lr_lds = stage1_lds_bytes(L[i].d_in, bt, chunk);
        // up to four tokens and a channel-major copy of S_r V_r^T: stage 1 reads only the dropped channels' rows
        const int parts = (L[i].rank + kTile - 1) / kTile;
        if (bt <= 4 && cfg[i].lowrank_wgs > 0 && L[i].rank > 0 && L[i].SVc && L[i].t_sum && parts <= cfg[0].waves && lowrank_copy_supported(L[i].d_in, L[i].rank)) {
            h.SVc = L[i].SVc;
            h.lr_wgs = std::min(cfg[i].lowrank_wgs, L[i].d_in / 8);
            // a wave's list (all of its channels at worst) has to fit: at least as many workgroups as keep the launch's LDS under 40 KiB
            while (direct_lds(h.cap_s1 = direct_cap(L[i].d_in, h.lr_wgs * cfg[0].waves), cfg[0].waves, bt) > 40 * 1024 && h.lr_wgs < L[i].d_in / 8) h.lr_wgs *= 2;
            lr_lds = direct_lds(h.cap_s1, cfg[0].waves, bt);
        }
        h.s1 = stage1_args(L[i], X, batch, cfg[i], h.lr_wgs, cfg[0].waves, chunk);
        h.L = L[i]; h.Y = Y[i];
        h.wait_polls = cfg[i].wait_polls > 0 ? cfg[i].wait_polls : kWaitLimitPolls;
        const int gather_wgs = cfg[i].tile_map == 2 ? ((tiles + 7) / 8) * 8 * cfg[i].splits : tiles * cfg[i].splits;
        if (cfg[i].tile_map != 2 && (unsigned long long)gather_wgs * tiles >= 1ull << 32) return hipErrorInvalidValue;   // (tiles_inv is exact below)
        h.X = (const uint16_t *)X; h.M = L[i].M; h.sync = L[i].sync; h.t_tag = L[i].t_tag; h.yacc = L[i].yacc; h.act_bits = L[i].act_bits;
        h.waves = cfg[0].waves;
        h.d_in = L[i].d_in; h.d_out = L[i].d_out; h.rank = L[i].rank; h.batch = batch;
        h.tiles = tiles; h.splits = cfg[i].splits; h.cap = direct_cap(L[i].d_in, R_all);
        h.tiles_inv = tiles == 1 ? 0u : (uint32_t)((1ull << 32) / tiles + 1);
        h.tile_map = cfg[i].tile_map; h.union_all = L[i].batch_mask_mode == 1; h.tau_ge = L[i].tau_ge;
        h.q_base = L[i].d_in / 8 / R_all; h.q_rem = L[i].d_in / 8 % R_all;
        h.u_base = L[i].rank / cfg[i].splits; h.u_rem = L[i].rank % cfg[i].splits;
        total += h.lr_wgs + gather_wgs;
        ga.wg_end[i] = total;
        const size_t need = direct_lds(h.cap, cfg[0].waves, bt);
        if (need > 64 * 1024) return hipErrorInvalidValue;
        lds = std::max(lds, need);
        if (lr_lds > 64 * 1024) return hipErrorInvalidValue;
        lds = std::max(lds, lr_lds);
    }
    for (int i = n; i < kMaxGroup; ++i) ga.wg_end[i] = total;
    ga.gate_up = gate_up ? 1 : 0;
    dim3 grid(total, 1, nz), block(kWave * cfg[0].waves);
    const bool nt = cfg[0].nontemporal != 0;
    bool ext = false;
    for (int i = 0; i < n; ++i) ext = ext || L[i].rules || L[i].bias || L[i].keep_signed;
    bool svc = false;
    for (int i = 0; i < n; ++i) svc = svc || ga.job[i].SVc;
#define RS_U3(DT, NT, EXT)                                                                                                          \
    do {                                                                                                                            \
        if (svc && BT <= 4) hipLaunchKernelGGL((k_rsparse_fused<DT, BT, NT, EXT, BT <= 4, 4>), grid, block, lds, stream, ga);      \
        else hipLaunchKernelGGL((k_rsparse_fused<DT, BT, NT, EXT, false, 4>), grid, block, lds, stream, ga);                       \
    } while (0)
#define RS_U(DT)                                                                                        \
    RS_DISPATCH_BT(bt, {                                                                                \
        if (nt && !ext) RS_U3(DT, true, false);                                                         \
        else if (nt) RS_U3(DT, true, true);                                                             \
        else if (!ext) RS_U3(DT, false, false);                                                         \
        else RS_U3(DT, false, true);                                                                    \
    })
    if (L[0].dtype == F16) { RS_U(F16) } else { RS_U(BF16) }
#undef RS_U
#undef RS_U3
    return hipGetLastError();
}

hipError_t launch_finish(const LayerView *L, int n, int batch, void *const *Y, bool use_rank, hipStream_t stream)
{
    if (!same_shape_class(L, n)) return hipErrorInvalidValue;
    const int bt = batch_tile(batch);
    const int nz = (batch + bt - 1) / bt;
    FinishGroupArgs ga{};
    ga.n = n;
    size_t lds = 16;
    int total = 0, max_passes = 0;
    for (int i = 0; i < n; ++i) {
        FinishArgs &a = ga.job[i];
        a.L = L[i]; a.Y = Y[i]; a.batch = batch;
        a.use_rank = use_rank ? L[i].rank : 0;
        const int chunks = (a.use_rank + 7) / 8;          // 16-byte pieces per row of U_r
        int lpr = 1;
        while (lpr < chunks && lpr < 64) lpr <<= 1;
        a.lpr = lpr;
        a.passes = chunks == 0 ? 0 : (chunks + lpr - 1) / lpr;
        max_passes = std::max(max_passes, a.passes);
        const int rows_per_wg = 4 * (64 / lpr) * kFinishGroups;
        total += (L[i].d_out + rows_per_wg - 1) / rows_per_wg;
        ga.wg_end[i] = total;
        lds = std::max(lds, (size_t)bt * a.use_rank * 4 + 16);
    }
    for (int i = n; i < kMaxGroup; ++i) ga.wg_end[i] = total;
    dim3 grid(total, 1, nz), block(256);
#define RS_F(DT)                                                                                           \
    RS_DISPATCH_BT(bt, {                                                                                   \
        if (max_passes <= 1) hipLaunchKernelGGL((k_finish<DT, BT, 1>), grid, block, lds, stream, ga);      \
        else if (max_passes == 2) hipLaunchKernelGGL((k_finish<DT, BT, 2>), grid, block, lds, stream, ga); \
        else hipLaunchKernelGGL((k_finish<DT, BT, 0>), grid, block, lds, stream, ga);                      \
    })
    if (L[0].dtype == F16) { RS_F(F16) } else { RS_F(BF16) }
#undef RS_F
    return hipGetLastError();
}

hipError_t launch_dense_axpy(const LayerView *L, const Launch *cfg, int n, const void *X, int batch, void *const *Y,
                             hipStream_t stream)
{
    if (!same_shape_class(L, n)) return hipErrorInvalidValue;
    const int bt = batch_tile(batch);
    const int nz = (batch + bt - 1) / bt;
    GroupArgs ga{};
    ga.n = n;
    size_t lds = 0;
    int total = 0;
    for (int i = 0; i < n; ++i) {
        GatherArgs &a = ga.job[i];
        const int tiles = (L[i].d_out + kTile - 1) / kTile;
        a.L = L[i]; a.X = (const uint16_t *)X; a.batch = batch; a.splits = cfg[i].splits; a.tiles = tiles;
        a.cap = gather_cap(L[i].d_in, cfg[i].splits);
        a.tile_map = cfg[i].tile_map;
        total += cfg[i].tile_map == 2 ? ((tiles + 7) / 8) * 8 * cfg[i].splits : tiles * cfg[i].splits;
        ga.wg_end[i] = total;
        lds = std::max(lds, gather_lds_bytes(L[i].d_in, cfg[i].splits, cfg[0].waves, bt));
    }
    for (int i = n; i < kMaxGroup; ++i) ga.wg_end[i] = total;
    dim3 grid(total, 1, nz), block(kWave * cfg[0].waves);
    const bool nt = cfg[0].nontemporal != 0;
#define RS_D(DT)                                                                                     \
    RS_DISPATCH_BT(bt, {                                                                             \
        if (nt) hipLaunchKernelGGL((k_dense_axpy<DT, BT, true>), grid, block, lds, stream, ga);      \
        else hipLaunchKernelGGL((k_dense_axpy<DT, BT, false>), grid, block, lds, stream, ga);        \
    })
    if (L[0].dtype == F16) { RS_D(F16) } else { RS_D(BF16) }
#undef RS_D
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_finish(L, n, batch, Y, false, stream);
}

// x = round16(silu(g) * u) written out (Sec. 3.1).  Forming it inside the gather kernel's own token loads was
// measured and lost: every workgroup scans the whole token, so the activation was evaluated ~400 times over
// (24.0 us against 22.1 us for this kernel followed by the plain layer, 11008 -> 4096).
template <int DT>
__global__ void k_gated_input(const uint16_t *G, const uint16_t *Up, uint16_t *out, size_t n8)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n8; i += stride) *reinterpret_cast<u32x4 *>(out + i * 8) = load_x8<DT>(Up, G, i * 8);
}

hipError_t launch_gated_input(const void *G, const void *Up, void *out, size_t n, int dtype, hipStream_t stream)
{
    if (n == 0 || (n % 8) != 0) return hipErrorInvalidValue;
    const size_t n8 = n / 8;
    size_t blocks = (n8 + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    if (dtype == F16)
        hipLaunchKernelGGL(k_gated_input<F16>, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint16_t *)G,
                           (const uint16_t *)Up, (uint16_t *)out, n8);
    else
        hipLaunchKernelGGL(k_gated_input<BF16>, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint16_t *)G,
                           (const uint16_t *)Up, (uint16_t *)out, n8);
    return hipGetLastError();
}

}  // namespace rsparse
