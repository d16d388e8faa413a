// Internal launch interface between the C-ABI host code (api.cpp) and the gfx950 kernels
// (kernels.hip).  Not installed; the public boundary is include/rsparse.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rsparse {

constexpr int kWave = 64;        // CDNA wavefront width
constexpr int kTile = 512;       // output columns per wave: 64 lanes x one 16-byte load (8 x 16-bit)
constexpr int kMaxBT = 8;        // tokens held in registers per workgroup (batch tile)
// Smallest batch that R-Sparse on layers with the operand-layout copy takes to the matrix cores by default (measured: the
// vector path wins up to 4 tokens: 4096 x 4096 18.8 us at four, 14.1 on the matrix cores at five, but 16.2 at two), and the
// smallest at which a dense kernel asked for by name gives way to them (the automatic choice: rsparse_dense_ref_group).
constexpr int kMfmaDefaultMinBatch = 5;
constexpr int kMfmaDefaultMinBatchDense = 2;

// Which channels of a token are kept (R-Sparse, Sec. 3.4: the sparsification function, and its fixed-count variant),
// in one form:  v >= ge  ||  (v == eq && channel <= cut),  with v = |x| (v = x for the signed threshold).
//   |x| >= t:   ge = t, eq = NaN (never equal).        |x| > t:  ge = the next fp32 above t.
//   fixed count k:  eq = the k-th largest magnitude of the token, ge = the next fp32 above it, cut = the last channel
//   among those equal to it that still belongs to the k (lower channels first).
struct KeepRule {
    float ge, eq;
    int cut, pad;
};

// Device-side view of one prepared layer plus its per-call scratch.
struct LayerView {
    const uint16_t *M;      // [d_in + rank][d_out]: W column-major (row c = W[:, c]), then U_r^T (row d_in + j = U_r[:, j])
    const uint16_t *SVt;    // [rank][d_in]  = S_r V_r^T
    const uint16_t *U;      // [d_out][rank] = U_r, row-major
    const uint16_t *SVc;    // [d_in][rank] channel-major copy of S_r V_r^T (row c = its column c), or nullptr
    float *t_sum;           // [nz][BT][rank] fp32 sums of the stage 1 that reads SVc; zero between calls (or nullptr)
    float *t;               // [nz][BT][rank] stage-1 result, fp32
    float *yacc;            // [max_batch][d_out] fp32 accumulators; zero between calls
    int32_t *act_list;      // [nz][d_in] ascending kept channels of batch tile z (union over its tokens)
    uint32_t *act_bits;     // [nz][d_in] per list entry: bit b = token b of the tile keeps it
    int32_t *act_count;     // [nz]
    int *sync;              // arrival counters (zero between calls) and generations of the one-launch kernels (layout: kSync* below)
    uint32_t *t_pub;        // [nz][BT][rank] one-launch 4-bit kernel: t as fp32 bits; all-ones (not ready) between calls (or nullptr)
    unsigned long long *t_tag;  // [t_slots][rank] one-launch kernels of 16-bit weights: {generation + 1 of the launch that wrote it, t as fp32 bits}
    int t_slots;            // token slots of t_tag (max_batch rounded up to whole batch tiles)
    // strip-major W for the strip kernel: strip s holds columns [s * strip_w, (s + 1) * strip_w) of all d_in + rank
    // rows (row c = W[:, c], row d_in + j = U_r[:, j]) contiguously, [strips][d_in + rank][strip_w]; columns past
    // d_out are zero
    const uint16_t *Ms;
    int strip_w;
    long long strip_stride; // 16-bit elements from one strip to the next: (d_in + rank + padding rows) * strip_w
    int32_t *act_seg;       // [nz][d_in / 8] strip kernel: kept channels found in each channel range of batch tile z
    // 4-bit weights (Mq != nullptr; then M is null).  A column tile is kQ4Tile = 1024 outputs: lane l
    // of a wave owns the 8 bytes T * 512 + l * 8 .. of a row, two words h = 0, 1; byte k of word h holds the
    // code of column T * 1024 + h * 512 + l * 8 + k in its low nibble and of column ... + 4 + k in its high one.
    const uint8_t *Mq;      // [d_in][qtiles * 512] bytes, row c = the codes of W[:, c]
    const uint16_t *qs;     // [d_in >> qshift][qtiles * 1024] group scales, 16-bit of dtype, plain column order
    const uint8_t *qz;      // [d_in >> qshift][qtiles * 1024] group zero points, one per byte
    const uint16_t *Ut;     // [rank][qtiles * 1024] = U_r^T, zero-padded rows (the one-launch 4-bit kernel streams it)
    int qshift, qtiles;     // log2(group size); column tiles of 1024
    int d_in, d_out, rank;
    int dtype, out_dtype, cmp_mode, batch_mask_mode;
    float tau;
    float tau_ge;           // the threshold as a KeepRule::ge (host-computed from tau and cmp_mode)
    int keep_signed;        // cmp_mode 2: the rule applies to x itself, not to |x|
    const KeepRule *rules;  // fixed-count activation: [batch] per-token rules written by launch_topk_rules; else nullptr
    const float *bias;      // [d_out] fp32 added to every token's output before the rounding, or nullptr
};

// Dense 4-bit baseline over row-major codes (kernels_q4row.hip): Qrow [d_out][d_in/2] (channel 2j in the low nibble of byte
// j), Srow / Zrow [d_out][d_in >> qshift].  Needs batch_tile * d_in * (2 + 1/8) bytes of LDS <= 64 KiB and groups >= 32.
bool q4_rowdot_supported(int d_in, int batch);
hipError_t launch_q4_dense_rowdot(const uint8_t *Qrow, const uint16_t *Srow, const uint8_t *Zrow, int qshift, int dtype, int out_dtype,
                                  int d_in, int d_out, const void *X, int batch, void *Y, hipStream_t stream);

// Fixed-count activation: per token of X [batch][d_in] the KeepRule that keeps exactly min(k, non-NaN channels)
// channels of largest magnitude (ties: lower channel first), for n layers that read X in one launch.
hipError_t launch_topk_rules(const void *X, int dtype, int batch, int d_in, const int *k, KeepRule *const *rules, int n, hipStream_t stream);

// What the matrix-core path holds of a layer beside LayerView (all null without it).  Operand layout of a matrix: [block of
// 16 rows][step of 32 columns][64 lanes][16 bytes], lane l of a tile = columns 8 (l / 16) .. + 7 of row l % 16; rows and
// columns past the matrix are zero.
struct MatrixView {
    const uint16_t *W, *SVt, *U;   // (W null: its part comes from an earlier launch, in yc)  W [d_out][d_in], S_r V_r^T [rank rounded up to 32][d_in], U_r [d_out][rank]
    void *t;                       // t: its 16-bit parts, then as it is; mfma_t_bytes(rank)
    float *t_acc;                  // fp32 sums of t, [32 tokens][rank rounded up to 32]; zero between calls
    int *t_flags;                  // [t_flag_words(rank)]; zero between calls
    float *yc;                     // [token tile][yc_rows][16 tokens] fp32 sums of the W part; zero between calls
    int yc_rows;
    int16_t keep_min;              // LayerView::tau_ge as the smallest kept 16-bit pattern of |x| (keep_signed: of x, as a two's complement number)
};

// Per-call scratch of a layer: what the kernels write besides Y.  Normally owned by the handle (allocated when the
// layer is prepared); rsparse_linear_static points it into a file-scope device array instead.
struct ScratchView {
    float *t, *yacc;
    int32_t *act_list;
    uint32_t *act_bits;
    int32_t *act_count, *act_seg;
    int *sync;
    uint32_t *t_pub;
    unsigned long long *t_tag;
    KeepRule *rules;
    int t_slots;
    size_t n_t, n_y, sync_n;       // 32-bit words of t / t_pub (and 64-bit words of t_tag), of yacc, of sync
};

// Limits of the static scratch (static_scratch.hip): one batch tile of up to 8 tokens, dimensions up to 32768,
// rank up to 2048 -- 1.6 MB carved out of a 2 MiB array.
constexpr int kStaticMaxBatch = 8, kStaticMaxDim = 32768, kStaticMaxRank = 2048;
// The scratch of one call in the calling device's static array (its address is looked up once per device), cleared
// for this call by one fill launch on `stream`: accumulators and counters zero, hand-off entries "not written".
// Allocates nothing.
hipError_t static_scratch_for_call(int device, int d_out, int rank, int batch, hipStream_t stream, ScratchView *out);

struct Launch {
    int splits;        // channel splits per column tile
    int waves;         // waves per workgroup (first launch / dense axpy)
    int lowrank_rows;  // rows of S_r V_r^T per stage-1 workgroup
    int lowrank_wgs;   // > 0: stage 1 of the one-launch kernel at up to four tokens reads the channel-major copy of S_r V_r^T
                       // (dropped channels' rows only) with this many workgroups, each on a fixed channel range
    int nontemporal;
    int tile_map;      // 1: tile-fastest workgroup order, 2: XCD-aware (a tile's splits share id mod 8)
    int wait_polls;    // one-launch kernel: bound on re-reads of an unpublished t entry; 0 = default
    int skip_stage1;   // one-launch kernel, test hook: stage 1 publishes nothing, so every wait runs out
};

// Arrival counters of the one-launch path, as offsets into LayerView::sync (32-bit words).  Every counter has a 128-byte line of
// its own: the memory system performs atomics on one line one after the other, whatever their words (256 workgroups that add
// to 8 tiles' sums, count their arrival and store, by itself: 6.6 us with the counters packed into one line, 4.2 with a line each).
constexpr int kSyncLine = 32;
constexpr int kSyncTilesDone = 0;              // one-launch 4-bit kernel: column tiles (over all batch tiles) whose outputs have been stored
constexpr int kSyncError = 1 * kSyncLine;      // set when a bounded wait ran out (results of that call are invalid)
constexpr int kSyncMaxZ = 4;                   // batch tiles per launch
// {counter, generation} (the hand-off of t, device_stage1.h), a line each:
constexpr int kSyncStage1 = 2 * kSyncLine;     // [kSyncMaxZ] per batch tile: stage-1 workgroups that have published their t, or (channel-major form) added their part of it
constexpr int kSyncTile = kSyncStage1 + kSyncMaxZ * kSyncLine;   // [nz][tiles]: channel splits of the column tile (strip) that have added their sums
__host__ __device__ inline int sync_tile(int tiles, int z, int tile) { return kSyncTile + (z * tiles + tile) * kSyncLine; }
inline size_t sync_words(int tiles, int nz) { return (size_t)kSyncTile + (size_t)(nz < kSyncMaxZ ? nz : kSyncMaxZ) * tiles * kSyncLine; }
// Matrix-core path, MatrixView::t_flags (32-bit words; every part starts a 128-byte line of its own): a flag per block of 16
// rank indices (its t is stored), an arrival counter per block (K slices), a line apart, kTReadSubs counters a line apart of the
// units of W that have read all of t, and how many of those counters are complete.
constexpr int kTReadSubs = 32;
__host__ __device__ inline int t_flag_pitch(int rank) { return (rank + 511) / 512 * 32; }
__host__ __device__ inline int t_arrival(int rank, int block) { return t_flag_pitch(rank) + block * kSyncLine; }
__host__ __device__ inline int t_read_at(int rank) { return t_arrival(rank, (rank + 31) / 32 * 2); }
inline size_t t_flag_words(int rank) { return (size_t)t_read_at(rank) + 32 * kTReadSubs + 32; }

// All launchers take a group of n <= kMaxGroupLayers layers that read the same input X (same d_in and
// dtype); cfg[0].waves and cfg[0].nontemporal apply to the whole launch.
constexpr int kMaxGroupLayers = 4;

// First launch: stage 1 of the low-rank part (with_t) and threshold + compaction + gather-GEMV over
// the kept columns into yacc (with_gather), as independent workgroups of one grid.
hipError_t launch_sparse_and_t(const LayerView *L, const Launch *cfg, int n, const void *X, int batch, bool with_t,
                               bool with_gather, hipStream_t stream);
// The whole layer in ONE launch: the stage-1 workgroups publish t, every gather workgroup also streams
// its share of the rows of U_r^T (as channels d_in.. with coefficients t), and the last workgroup to
// arrive at a column tile rounds and stores that tile of Y.  cfg[i].splits must satisfy
// direct_lds_bytes(d_in, splits, waves, bt) <= 64 KiB.
// gate_up: L[0], L[1] are the gate and up projections of an MLP (same d_out, out_dtype == dtype); the kernel
// stores H = round(silu(round(g)) * round(u)) to Y[0] instead of the two outputs (Y[1] is not written).
hipError_t launch_fused(const LayerView *L, const Launch *cfg, int n, const void *X, int batch, void *const *Y,
                        hipStream_t stream, bool gate_up = false);
// First launch of a layer with 4-bit weights (batch tiles of at most 4 tokens): as launch_sparse_and_t, with the codes
// dequantised in registers -- per quantisation group the kernel accumulates sum_c x_c q_c and sum_c x_c and
// applies scale and zero point once, when the group ends.  dense: every channel is kept (the dense baseline
// on the same weights).  Y_fused == nullptr: launch_finish completes the layer.  Y_fused != nullptr: the whole
// layer in this one launch, as launch_fused (not with dense).
constexpr int kQ4Tile = 1024;
// (one layer); n layers that read the same input share a launch of the first kind.
hipError_t launch_q4(const LayerView *L, const Launch *cfg, int n, const void *X, int batch, bool with_t, bool dense,
                     void *Y_fused, hipStream_t stream);
// Second launch: Y = round(yacc + U_r t) (use_rank) or round(yacc); re-zeroes yacc.
hipError_t launch_finish(const LayerView *L, int n, int batch, void *const *Y, bool use_rank, hipStream_t stream);
// Dense baselines.
hipError_t launch_dense_axpy(const LayerView *L, const Launch *cfg, int n, const void *X, int batch, void *const *Y,
                             hipStream_t stream);
// Row dots over the operand-layout copy of W (MatrixView::W), a batch of up to 8 tokens per tile within 64 KiB of LDS.
hipError_t launch_dense_rowdot(const LayerView *L, const MatrixView *M, const Launch *cfg, int n, const void *X, int batch, void *const *Y,
                               hipStream_t stream);
// Matrix-core path for up to 32 tokens over the row-major copy of W: n layers that read the same input in one launch.
// chan_bits[i] [d_in] receives, per channel, the bit mask of the tokens that keep it.  phases: 3 = the whole call (t is
// handed over inside the launch through t_flags); 1 = t only, 2 = the rest, as launches of their own.
// dense = the dense product Y = X W^T through the same kernel (no masks, no low-rank part).
bool mfma_path_supported(const MatrixView &M, int batch);
size_t mfma_t_bytes(int rank);
// A row-major matrix [rows][cols] (device; cols a multiple of 8) in operand layout, rows padded to row_pad (16 or 32).
size_t mfma_operand_bytes(size_t rows, size_t cols, size_t row_pad);
hipError_t launch_pack_operand(const uint16_t *src, size_t rows, size_t cols, size_t row_pad, uint16_t *dst, hipStream_t stream);
// dst [cols][ld >= rows] = transpose of src [rows][cols], 16-bit, all multiples of 8 (device).
hipError_t launch_transpose16(const uint16_t *src, size_t rows, size_t cols, uint16_t *dst, size_t ld, hipStream_t stream);
hipError_t launch_mfma(const LayerView *L, const MatrixView *M, int n, const void *X, int batch, void *const *Y, uint32_t *const *chan_bits, int cus,
                       int phases, bool dense, int wait_polls, int skip_stage1, hipStream_t stream);
// 4-bit weights on the matrix cores (kernels_mfma_q4.hip), up to 32 tokens, n layers that read the same input: adds the W
// part of each layer (dense: the whole product) to its yc, [token tile][qtiles * 1024][16 tokens], and stores t in fp32, as
// launch_mfma's phase 2 expects it of such layers (MatrixView::W null), which completes them.
int mfma_t_slices(int t_blocks, int d_in, int nw, int cus);
hipError_t launch_mfma_q4(const LayerView *L, const MatrixView *M, int n, const void *X, int batch, bool dense, int cus, hipStream_t stream);
// The same over column-major W (kernels_mfma_cols.hip; layers without the operand-layout copy), n layers that read the same
// input: yc [token tile][yc_rows >= d_out][16 tokens].
hipError_t launch_mfma_cols(const LayerView *L, const MatrixView *M, int n, const void *X, int batch, bool dense, int cus, hipStream_t stream);
// The whole layer over strip-major weights (LayerView::Ms), up to 8 tokens per batch tile: one workgroup per strip
// of strip_w output columns streams all kept rows of the strip and stores its slice of Y (cfg[i].splits == 1), or
// `splits` workgroups per strip meet in yacc.  fused: stage 1 runs in the same launch and hands t over through
// LayerView::t_tag; otherwise t must have been stored to LayerView::t by an earlier launch
// (launch_sparse_and_t with with_gather = false).  dense: the dense product Y = X W^T through the same kernel
// (every channel kept, no low-rank part).  Layers of a group share d_in, dtype and strip_w.
hipError_t launch_strip(const LayerView *L, const Launch *cfg, int n, const void *X, int batch, void *const *Y,
                        bool fused, bool dense, int cus, hipStream_t stream);
// Stamps builds only (see device_stage1.h): where the waves of the one-launch kernels write their phase time stamps;
// hipErrorNotSupported in product builds.
hipError_t set_stamp_buffer(void *buf_dev, int capacity_waves);
hipError_t set_stamp_buffer_columns(void *buf_dev, int capacity_waves);      // (of kernels.hip, for set_stamp_buffer)
int strip_waves(int batch);                       // waves per workgroup the strip kernel runs with
// list entries per wave that fit in LDS for this launch shape; 0 = the shape does not fit (more splits needed)
int strip_list_cap(int d_in, int rank, int splits, int waves, int bt, int strip_w);
bool strip_width_ok(int w);
// out[0:n) = round16(silu(G) * Up), n a multiple of 8, all 16-byte aligned.
hipError_t launch_gated_input(const void *G, const void *Up, void *out, size_t n, int dtype, hipStream_t stream);
size_t gather_lds_bytes(int d_in, int splits, int waves, int bt, int fused_rank = 0);
size_t direct_lds_bytes(int d_in, int splits, int waves, int bt);   // launch_fused's gather workgroups
bool direct_supported(int d_in, int d_out, int rank);               // launch_fused: M within its buffer descriptor (2 GiB less 16 MiB)
bool lowrank_copy_supported(int d_in, int rank);                    // ... and the channel-major copy within its own
size_t lowrank_lds_bytes(int d_in, int bt);
// Stage 1 of the one-launch kernels with `rows` rows of S_r V_r^T per workgroup: channels of the token(s) staged in LDS at a time, 0: none.
int stage1_chunk(int d_in, int bt, int rows, int unstaged);
size_t stage1_lds_bytes(int d_in, int bt, int chunk);
bool rowdot_supported(int d_in, int batch);

}  // namespace rsparse
