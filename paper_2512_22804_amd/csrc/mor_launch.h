// Host-side launch interface between the C ABI (mor_api.hip) and the kernels (mor_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace mor {

// Device pointers of one call, passed to kernels by value.
struct KOut {
    uint8_t*  fp8;      int64_t ld_fp8;
    uint16_t* bf16;     int64_t ld_bf16;     // bf16 == nullptr: no fallback payload is written
    float*    scale;
    float*    amax;
    float*    err_sum;
    uint32_t* nnz;
    uint8_t*  mask;
    float*    err5_sum;
    uint8_t*  e8m0;     // [P] biased exponents of the applied scales (GAM / E8M0 scaling), may be nullptr
    uint32_t* gmant;    // [2] fraction bits of the group mantissas (E4M3, E5M2), may be nullptr
    float*    amin;     // [P] smallest non-zero magnitude of blocks that failed M_1 (three-way recipe), may be nullptr
    uint16_t* fake;     // fake quantization: de-quantized BF16 output instead of the FP8 payload (then bf16 == fake
    int64_t   ld_fake;  //   so that BF16 blocks pass through); nullptr otherwise
};

struct KShape {
    int64_t rows, cols, ld;
};

// Block grid of an operand: nominal block pr x pc, grid gr x gc (edge blocks smaller when ragged).
struct StatsGeom {
    int64_t rows, cols, pr, pc, gc;
    int32_t uniform;        // 1: every block has pr * pc elements
};
enum { kGranTensor = 0, kGranSub = 1, kGranBlock = 2, kGranRow = 3, kGranCol = 4, kGranSubCol = 5, kGranBlock64 = 6 };
inline StatsGeom make_geom(int gran, int64_t rows, int64_t cols) {
    StatsGeom g{rows, cols, rows, cols, 1, 1};
    switch (gran) {
    case kGranSub:     g.pr = 1;   g.pc = 128; break;
    case kGranBlock:   g.pr = 128; g.pc = 128; break;
    case kGranRow:     g.pr = 1;   g.pc = cols; break;
    case kGranCol:     g.pr = rows; g.pc = 1;  break;
    case kGranSubCol:  g.pr = 128; g.pc = 1;   break;
    case kGranBlock64: g.pr = 64;  g.pc = 64;  break;
    default: break;
    }
    g.gc = (cols + g.pc - 1) / g.pc;
    g.uniform = (rows % g.pr == 0 && cols % g.pc == 0) ? 1 : 0;
    return g;
}
inline int64_t geom_parts(const StatsGeom& g) { return ((g.rows + g.pr - 1) / g.pr) * g.gc; }

// Shift that takes a row or column, held in `bits` bits, to its block of a dimension of `dim` elements.  One block that spans the
// dimension need not be a power of two: shifting out all but the sign bit leaves 0 for every non-negative index.
inline int block_shift(int64_t block, int64_t dim, int bits) {
    if (block >= dim) return bits - 1;
    int l = 0;
    while ((1ll << l) < block) ++l;
    return l;
}
// Reciprocal of d (1 <= d < 2^31) for n / d == mulhi(2n, mul) >> shift, n < 2^31: with l = ceil(log2 d) and
// mul = floor(2^(31+l) / d) + 1, mul * d exceeds 2^(31+l) by at most d <= 2^l, so the quotient is off by less than 1 / d.
inline void recip_of(int64_t d, uint32_t* mul, uint32_t* shift) {
    uint32_t l = 0;
    while ((1ll << l) < d) ++l;
    *mul = (uint32_t)((1ull << (31 + l)) / (unsigned long long)d + 1ull);
    *shift = l;
}
// Leading dimensions up to which the kernels for padded rows form 32-bit byte offsets inside a tile, and the same for the tile's
// span (`rows` of the longest row); beyond them the general paths are taken.
constexpr int64_t kRowMapMaxLd = 1 << 22;
inline int64_t longest_row(const KShape& sh, const KOut& o) {
    int64_t ld = sh.ld;
    if (o.fp8 && o.ld_fp8 > ld) ld = o.ld_fp8;
    if (o.bf16 && o.ld_bf16 > ld) ld = o.ld_bf16;
    if (o.fake && o.ld_fake > ld) ld = o.ld_fake;
    return ld;
}
inline bool row_map_fits(int64_t ld, int64_t rows) { return ld < kRowMapMaxLd && rows * ld * 2 < 0x7FFFFFFFll; }

// Workspace layout for the passes that need one (all offsets 16-byte aligned).
struct TensorPlan {
    int     amax_blocks;     // grid of the amax pass
    int64_t quant_blocks;    // grid of the quantize pass
    size_t  off_amax_part;   // uint32[amax_blocks]
    size_t  off_err_part;    // float[quant_blocks]
    size_t  off_err5_part;   // float[quant_blocks]
    size_t  off_nnz_part;    // uint32[quant_blocks]
    size_t  off_decision;    // uint32[4]: [0] global amax bits
    size_t  off_flush_part;  // uint32[amax_blocks]
    size_t  bytes;
};
TensorPlan plan_tensor(int64_t rows, int64_t cols);
size_t scope_workspace_bytes(int64_t n_part);

constexpr int kProfMax = 16;
// Optional per-kernel timing: when non-null, start[i]/stop[i] are recorded around the i-th kernel.
struct KProf {
    int32_t capacity;
    int32_t count;
    hipEvent_t start[kProfMax];
    hipEvent_t stop[kProfMax];
    int32_t kernel[kProfMax];
};
enum KernelId {
    kKernSub1x128 = 1, kKernBlock128 = 2, kKernTensorAmax = 3, kKernTensorQuant = 4, kKernTensorFinalize = 5,
    kKernFallbackCopy = 6, kKernScopeReduce = 7, kKernScopeDecide = 8, kKernScopeFillMask = 9,
    kKernStatsPartial = 10, kKernStatsFinal = 11, kKernGroupAmax = 12, kKernGroupMantissa = 13,
    kKernTeamBlock = 14, kKernColumnTile = 15, kKernColumnCombine = 16, kKernTensorStream = 17, kKernTeamStream = 18, kKernStreamClear = 19
};

// Records the caller's events around one kernel launch when profiling is requested.
struct ProfScope {
    KProf* prof; hipStream_t st; int slot;
    ProfScope(KProf* p, int kernel_id, hipStream_t s) : prof(p), st(s), slot(-1) {
        if (prof && prof->count < prof->capacity && prof->count < kProfMax) {
            slot = prof->count++;
            prof->kernel[slot] = kernel_id;
            (void)hipEventRecord(prof->start[slot], st);
        }
    }
    ~ProfScope() { if (slot >= 0) (void)hipEventRecord(prof->stop[slot], st); }
};

// Residency caps: bytes of dynamic LDS a launch reserves (and never touches) so that only 3 or 5 workgroups of 256
// lanes fit the 160 KB of a compute unit.  The streaming passes run faster with FEWER workgroups in flight than
// their register use would allow (measured on MI355X: pass B of the per-tensor path over several operands, whole layer call,
// 413.5 us at 3 per unit, 417 us at 4, 419 us at 5 and uncapped; the 128x128 team kernel 114 us at 4 or 5 against 116 us at 7; the quantize pass of the per-channel columns 0.609 ms per twelve-operand pass at 4 against 0.620 ms
// uncapped): fewer concurrent streams keep the accesses of each HBM channel closer together.  Kernels that need many
// waves to hide latency (de-quantization, 128x1 sub-columns) lose with a cap and have none.
constexpr int kResidency3 = 52000;
constexpr int kResidency4 = 39000;
constexpr int kResidency5 = 31000;

constexpr int kBatchMax = 64;     // operands per batch call

// Operands that are read twice (amax first, then quantize).  The first pass reads them without the non-temporal hint, so that
// they stay in the Infinity Cache (256 MB) for the second one, and a batch takes per-tensor operands and most of those under GAM
// scales in parts of at most kKeepGroupBytes, both passes of one part before the next part's.  Measured with bare passes (2 bytes
// read; 2 read and 3 written per element): 64 MB 39 -> 32 us, 224 MB 135 -> 114, 480 MB 295 -> 260 in one part and 228 in two,
// 960 MB 597 -> 566 in one.  The first pass itself is up to 15 % slower that way (6.0 instead of 7.0 TB/s), which an operand far
// larger than the cache does not get back: above kKeepMaxBytes the hint stays (pre-passes of GAM scaling and column amax).
constexpr int64_t kKeepGroupBytes = 256ll << 20;
constexpr int64_t kKeepMaxBytes = 1ll << 30;
// Per-tensor operands, whose quantize pass may also write a BF16 copy, keep kKeepTensorBytes of a part at any size: the same share
// of each of its operands, at the operand's end.  More pays in calls that follow each other (224 MiB falling back to BF16, us per
// call: none 146.4, 64 MiB 138, 96 MiB 134.8, 128 MiB 132.2, all 128.9; the six gradients of a layer 429, 412, 407.9, 406.6, 408), but a
// call whose output buffers have just been filled by others finds their unwritten lines in the cache and has them evicted: 179,
// 184.6, 185.8, 188.9, 203 us for its first pass.
constexpr int64_t kKeepTensorBytes = 96ll << 20;
inline bool keep_for_second_pass(const KShape& sh) { return sh.rows * sh.cols * 2 <= kKeepMaxBytes; }

// One operand of a batch (validated by the caller).
struct BatchItem {
    KShape sh;
    KOut o;
    const uint16_t* x;
    int gran, crit, scope;
    int scaling;            // 0 FP32 amax, 1 GAM, 2 E8M0 only
    int three;              // 1: type list [E4M3, E5M2, BF16]
    int ragged;             // 1: edge blocks may be smaller
    int lean;               // 1: the FP8 payload of blocks already known to stay in BF16 need not be written
    float th;
    void* stats;            // device mor_stats* or nullptr
    int64_t group_rows;     // GAM: 0 = one group (the whole operand); else the groups of Algorithm 1 are bands of this many rows
    int polls;              // how often a workgroup of a lone per-tensor operand looks for the decision before it leaves its tile to another
};
constexpr int kOnePolls = 1024;      // about half a millisecond
// Where such a call with the workspace of one operand keeps the words of the workgroups that left (for tests): bytes from its start, words.
struct LeftWords {
    size_t offset;
    int count;
};
LeftWords lone_tensor_left_words();
size_t batch_workspace_bytes(const BatchItem* items, int n);
hipError_t launch_batch(const BatchItem* items, int n, float near_tol, void* ws, size_t ws_bytes, hipStream_t st, KProf* prof);

// mor_partitions.hip: team kernels (64x64, per-channel rows, general 128x128) and column kernels
enum { kCritEq2 = 0, kCritEq3 = 1 };

// That many elements certain to flush (each contributes exactly 1 to the error sum of Eq. 2) prove "mean relative error
// >= th" for a block of `n` elements, whatever the other terms are: the 1 % margin over th * n covers the rounding of the
// binary32 error sums that the decision itself is taken from.  Only used for 0 < th < 0.9.
inline unsigned long long flush_need_of(float th, int64_t n) { return (unsigned long long)(1.01 * (double)th * (double)n) + 1ull; }

// Tensor-level decision (Section 3.1) over GAM-scaled sub-tensor blocks (128 x 128, 64 x 64, per-channel rows, 1 x 128 sub-rows,
// 128 x 1 sub-columns): the amax pre-pass of Algorithm 1 can prove the BF16 decision under Eq. 2 from elements that are certain to
// flush inside their block, so the block kernel writes the BF16 payload from its registers and the operand is not read a third time.
inline bool scope_proof_applies(const BatchItem& it) {
    // (fake quantization: o.bf16 == o.fake, and a proven operand's output is its input)
    if (it.scaling != 1 || it.scope != 1 || it.crit != kCritEq2 || it.three || it.o.bf16 == nullptr || it.group_rows != 0) return false;
    if (!(it.th > 0.0f && it.th < 0.9f)) return false;      // the flush count is compared with 1.01 * th * N + 1
    const bool whole_tiles = it.sh.rows % 128 == 0 && it.sh.cols % 128 == 0;
    if (it.gran == kGranBlock || it.gran == kGranBlock64 || it.gran == kGranSubCol) return whole_tiles;
    if (it.gran == kGranSub)      // the flat 1 x 128 kernel only (dense operand)
        return whole_tiles && it.sh.ld == it.sh.cols && it.o.ld_bf16 == it.sh.cols && (it.o.fake != nullptr ? it.o.ld_fake == it.sh.cols : it.o.ld_fp8 == it.sh.cols);
    return it.gran == kGranRow;
}
// Work units of the pre-pass (16384 elements each) and its per-operand arguments: per workgroup the largest amax and
// the number of certain flushes it saw.
inline int64_t scope_proof_units(const BatchItem& it) {
    if (it.gran == kGranRow) return (it.sh.rows * ((it.sh.cols + 4095) / 4096) + 3) / 4;
    return (it.sh.rows / 128) * (it.sh.cols / 128);
}
enum { kProveKindBlock128 = 0, kProveKindRows = 1, kProveKindBlock64 = 2, kProveKindSubRow = 3, kProveKindSubCol = 4 };
inline int scope_proof_kind(const BatchItem& it) {
    switch (it.gran) {
    case kGranRow: return kProveKindRows;
    case kGranBlock64: return kProveKindBlock64;
    case kGranSub: return kProveKindSubRow;
    case kGranSubCol: return kProveKindSubCol;
    default: return kProveKindBlock128;
    }
}
struct BlockProveItem {
    const uint16_t* x;
    int64_t rows, cols, ld;
    uint32_t* amax_part;     // [n_wg]
    uint32_t* flush_part;    // [n_wg]
    int n_wg;
    int kind;                // kProveKind*
    int keep;                // keep_for_second_pass
};
hipError_t launch_block_amax_prove(const BlockProveItem* ops, int n, hipStream_t st);

constexpr int kTeamKinds = 5;      // team kinds are numbered 0 .. kTeamKinds - 1 (mor_partitions.hip)
int team_kind_of(const BatchItem& it);
struct TeamRiders;      // mor_sub1x128.h
hipError_t launch_team_items(const BatchItem* items, const int* idx, int cnt, int kind, int crit, const uint32_t* const* gam_of,
                             TeamRiders* riders, hipStream_t st, KProf* prof);
hipError_t launch_subcol_items(const BatchItem* items, const int* idx, int cnt, int crit, const uint32_t* const* gam_of,
                               hipStream_t st, KProf* prof);
// Operands under GAM scales whose two passes share a launch, several in a call.
struct TeamStreamItem {
    const BatchItem* it;
    uint32_t* gam;           // the operand's mantissa words
    uint32_t* sync;          // [kStreamWords]
};
constexpr int kStreamWords = 2 * 8192;      // what the workspace has for the partials of the operand's pre-pass otherwise
int team_stream_kind(const BatchItem& it);      // operands of one number may share a launch; -1: not streamed
// Which calls stream them: from four operands and 8 MiB on all (us per call, launch by launch in parts / streamed: layer of twelve operands, fake
// quantization under a tensor-level decision, 8192 tokens x hidden 4096 498 / 430 at 128 x 128, 521 / 438 at 64 x 64, 506 / 444 by rows; 1024 x 2048 122 / 111,
// 123 / 113, 171 / 153; 512 x 1024 42.7 / 41.9, 47.3 / 45.6, 80 / 65; 64 x 256, of which some have ragged blocks and stay launch by launch, 34.2 / 34.8,
// 30.7 / 35.9).  Fewer have nobody to share the launch with, so it saves a launch and fills the gap between the passes, but at 128 x 128 takes about
// 2 us more to tell: 4096 x 4096 26.0 / 28.4, 8192 x 4096 40.5 / 40.5, 8192 x 14336 110.6 / 101.8; at 64 x 64 2048 x 4096 24.0 / 23.9, 4096 x 4096 30.7 / 27.3,
// 8192 x 4096 46.3 / 40.3; by rows 22.5 / 23.3, 26.7 / 26.0, 43.3 / 38.4.  (Two or three of more than 256 MiB together
// would gain too, but stay in parts: the interface promises no sequence of launches, but tests/test_gpu_launch_counts.py counts these.)
// Where other operands of the call have a pre-pass of their own (`beside`), streaming adds launches to theirs: layer with weights at 128 x 128,
// activations at 1 x 128 and gradients per tensor under GAM scales, 512 x 1024 55 / 66, 2048 x 1024 52 / 62, 1024 x 2048 (110 MB of weights) 131 / 133, 4096 x 2048
// 147 / 146, 4096 x 3072 (248 MB) 298 / 278.
inline bool stream_pays(int n, int64_t bytes, bool block128, bool beside) {
    if (n >= 4) return bytes >= (beside ? 128ll : 8ll) << 20;
    return bytes >= (block128 ? 128ll : 32ll) << 20 && bytes <= 256ll << 20;
}
hipError_t launch_team_stream_items(const TeamStreamItem* ops, int n, hipStream_t st, KProf* prof);
size_t column_workspace_bytes(int64_t rows, int64_t cols);
// Per-channel columns with a tensor-level decision: the column-amax pass counts certain flushes per column anyway, and their
// total may prove the operand's BF16 decision (Eq. 2); the quantize pass then writes the fallback and the word below says so.
inline bool column_tensor_proof_applies(const BatchItem& it) {
    return it.gran == kGranCol && it.scope == 1 && it.crit == kCritEq2 && !it.three && it.o.bf16 != nullptr && it.o.fake == nullptr &&
           it.th > 0.0f && it.th < 0.9f;
}
// Workgroups of the decision / mask / copy launch of a tensor-level decision, shared by its operands in proportion to their size.
// 1024 copy one operand as fast as it goes (8192 x 14336: 145.8 us per call, 145.3 at 4096) and are cheaper where nothing is copied
// (the same operand kept in E4M3: 70.5 against 73.2 us).  Several operands that no pre-pass can prove share them, and those that are
// copied get too few: a layer of twelve at 128 x 128, six of them copied, 475 us per call at 1024, 458 at 2048, 450 at 4096 (306
// against 308 us at 1 x 128, where none is copied).  A workgroup keeps at least four 16 KB tiles.
inline int scope_copy_budget(int n_unproven, int64_t unproven_bytes) {
    int64_t v = unproven_bytes >> 16;
    const int64_t cap = n_unproven < 4 ? 1024 * n_unproven : 4096;
    if (v > cap) v = cap;
    return (int)(v < 1024 ? 1024 : v);
}
// Per-channel columns: what the quantize pass has left of each strip, [n_strips x cols_padded], and the columns' amax.
struct ColumnSums {
    const float* err; const float* err5; const uint16_t* zero; const float* amax;
    int64_t cols_padded;
    int32_t n_strips;        // 0: the block kernels have left the blocks' sums already
};
// A column's strips are read one after another (eight or sixteen loads in flight), so what a lane has to read sets the time of the step that
// reads them where an operand is tall.  us per call, FP32 scales, weights:
// Sums of a tensor-level decision, in its reduce pass / by a launch of their own before it: 8192 x 512 (64 strips) 24.4 / 25.6, 12288 x 256
// (96) 27.6 / 28.1, 14336 x 256 (112) 29.7 / 29.5, 16384 x 128 (128) 30.9 / 29.9, 32768 x 128 (256) 44.1 / 39.6.
constexpr int kStripsInReduce = 96;
// Scales, by every workgroup of the quantize pass / by a launch of their own, which has nobody to share the reads with but costs a launch:
// up to 128 strips the former takes less (32768 x 1024 59.6 / 61.3); beyond, it depends on how many workgroups repeat the reads, and on
// whether the launch reads the flush counts of single columns as well: 65536 x 128 (512 workgroups) 63.1 / 65.8, 65536 x 256 (1024) 85.8 / 76.2,
// with flush counts 83.6 / 91.3, 131072 x 128 139 / 145; two of 200000 x 128 with flush counts (1564) 175 / 154.
inline bool column_scales_folded(int64_t n_strips, int64_t launch_workgroups, bool flush_counts) {
    return n_strips <= 128 || launch_workgroups <= (flush_counts ? 1024 : 512);
}
ColumnSums column_sums_of(const char* column_workspace, int64_t rows, int64_t cols, const float* amax);
uint32_t* column_tensor_proven_word(char* column_workspace, int64_t rows, int64_t cols);
// Per-channel rows that go along with per-channel columns, the operands of linear layers.
constexpr int kPairMax = 4;
struct PairRows {
    TeamStreamItem ops[kPairMax];      // (without GAM scales: no words)
    int n;
};
bool pair_takes_row(const BatchItem& it);
bool columns_pair(const BatchItem* items, const int* idx, int cnt);
hipError_t launch_channel_col_items(const BatchItem* items, const int* idx, int cnt, int crit, const uint32_t* const* gam_of,
                                    char* const* ws_of, const PairRows* rows, hipStream_t st, KProf* prof);

// One operand of a de-quantize batch (validated by the caller).
struct DeqItem {
    StatsGeom geom;
    const uint8_t* fp8; int64_t ld_fp8;
    const float* scale; const uint8_t* mask;
    const uint16_t* bf16; int64_t ld_bf16;
    uint16_t* y; int64_t ld_y;
    const uint8_t* e8m0; const uint32_t* gmant;
    int64_t group_rows;      // stored GAM form: rows per group (0 = one group)
};
hipError_t launch_dequantize_batch(const DeqItem* items, int n, hipStream_t st);
hipError_t launch_select_stats(const StatsGeom& geom, const float* err_sum, const uint32_t* nnz,
                               const uint8_t* mask, float th, float near_tol, void* out_dev, hipStream_t st);
hipError_t launch_histogram_update(uint32_t* hist, const void* stats_dev, int clear, hipStream_t st);

}  // namespace mor
