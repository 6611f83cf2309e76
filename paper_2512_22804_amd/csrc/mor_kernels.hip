// HIP kernels of the MoR analyse-select-quantize path for gfx950 (MI355X), and their launchers.
//
// One fused HBM pass per operand for sub-tensor granularities: 128-bit BF16 loads, integer amax,
// one IEEE division per block, hardware OCP-E4M3 conversion, relative-error reduction, decision
// (Algorithm 2 with [E4M3, BF16]) and emission, all from registers.  Per-tensor granularity needs
// the global amax before anything can be scaled and therefore reads the operand twice.
// The path is HBM-bound: there is no contraction in it, so no MFMA.
#include <type_traits>

#include "mor_device.h"
#include "mor_launch.h"
#include "mor_stream.h"
#include "mor_sub1x128.h"
#include "mor_team.h"

namespace mor {


// ======================================================================================
// 1 x 128 sub-channel blocks (Section 3: sub-channel partition; DeepSeek-style activations)
// A 16-lane DPP row owns one block at a time (16 lanes x 8 elements); a wave works on 4 blocks
// per load instruction and keeps 4 loads in flight, so every reduction stays inside a row.
// ======================================================================================
// One block per 16-lane row, 8 elements per lane.  `valid` is false for lanes beyond the last column of a
// ragged tensor (they hold zeros and store nothing).  FAKE: the de-quantized values go to dst_fake instead
// of the codes to dst_fp8.  `three`: the block may end in E5M2 (Section 3.2, three-way recipe).
template <int CRIT, bool DEFER, bool FAKE>
__device__ __forceinline__ void sub_block_body(const u32x4& raw, const uint16_t* __restrict__ src, bool valid, int l, int64_t p,
                                               const KOut& o, uint8_t* __restrict__ dst_fp8, uint16_t* __restrict__ dst_bf16,
                                               uint16_t* __restrict__ dst_fake, float th, uint32_t mode, uint32_t mg, uint32_t mg5,
                                               bool three) {
    Scan8 sc{0u, 0u};
    scan8(raw, sc);
    const uint32_t abits = row_allmax_u32(fold_max16(sc.amax2));
    float s = block_scale(abits, kE4M3Max, mode, mg);
    const float s5 = block_scale(abits, kE5M2Max, mode, mg5);
    const bool fast = abits < fast_amax_limit(mode);
    auto quantize = [&](auto fmt, float sc_, bool emit) -> float {
        constexpr bool E5 = decltype(fmt)::value;
        const float s_inv = FAKE ? 1.0f / sc_ : 0.0f;
        float e0 = 0.0f, e1 = 0.0f;
        if (fast) {
            u32x4 deq;
            const u32x2 codes = quant8_fast_deq<E5, FAKE>(raw, sc_, s_inv, e0, e1, deq);
            if (emit && valid) {
                if constexpr (FAKE) store16(dst_fake, deq);
                else store8(dst_fp8, codes);
            }
        } else if (valid) {
            e0 = quant8_careful_mem<E5>(src, sc_, emit && !FAKE ? dst_fp8 : nullptr, emit && FAKE ? dst_fake : nullptr, s_inv);
        }
        return e0 + e1;
    };
    float err = row_allsum_f32(quantize(std::false_type{}, s, true));
    float err5 = 0.0f;
    if constexpr (CRIT == kCritEq3) err5 = row_allsum_f32(quantize(std::true_type{}, s5, false));
    const uint32_t nnz = 128u - row_allsum_u32(fold_add16(sc.zero2));
    if (abits >= kInfBits) { err = __builtin_inff(); err5 = __builtin_inff(); }
    uint32_t mask = 0u;
    if constexpr (!DEFER) mask = (CRIT == kCritEq3) ? decide_eq3(err, err5) : decide_eq2(err, nnz, th);
    uint32_t amin_bits = 0u;
    if (three) {                                              // uniform over the launch
        const uint32_t mn = ~row_allmax_u32(~fold_min16(min_nonzero_m1(raw, 0xFFFFFFFFu))) & 0xFFFFu;
        if (mask == 1u) {
            amin_bits = nnz ? mn + 1u : 0u;
            if (range_fits_e5m2(abits, amin_bits, nnz)) {
                mask = 2u;
                s = s5;
                (void)quantize(std::true_type{}, s5, true);   // the E5M2 payload replaces the E4M3 one
            }
        }
    }
    if (l == 0) {
        o.scale[p] = s;
        o.amax[p] = __uint_as_float(abits << 16);
        o.err_sum[p] = err;
        o.nnz[p] = nnz;
        if constexpr (CRIT == kCritEq3) o.err5_sum[p] = err5;
        if constexpr (!DEFER) o.mask[p] = (uint8_t)mask;
        if (mode != kScaleFp32 && o.e8m0) o.e8m0[p] = (uint8_t)(__float_as_uint(s) >> 23);
        if (three && o.amin) o.amin[p] = __uint_as_float(amin_bits << 16);
    }
    if constexpr (!DEFER) {
        if (mask == 1u && dst_bf16 && valid) store16(dst_bf16, raw);
    }
}

// General 1 x 128 kernel (padded leading dimensions, ragged last column block, three types, fake
// quantization): grid.x = 128-column block, grid.y strides over groups of 16 rows.
template <int CRIT, bool DEFER, bool FAKE>
__global__ __launch_bounds__(256) void k_sub1x128_strided(const uint16_t* __restrict__ x, KShape sh, KOut o, float th,
                                                          uint32_t mode, const uint32_t* __restrict__ gam, uint32_t three, uint32_t group_rows) {
    const int lane = threadIdx.x & 63, g = lane >> 4, l = lane & 15;
    const int64_t cb = blockIdx.x, cpr = (sh.cols + 127) / 128;
    const int64_t c = cb * 128 + l * 8;
    const bool valid = c < sh.cols;
    if (mode == kScaleE8M0 && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) zero_group_mantissa(o.gmant);
    for (int64_t r = (int64_t)blockIdx.y * 16 + (threadIdx.x >> 6) * 4 + g; r < sh.rows; r += (int64_t)gridDim.y * 16) {
        const uint16_t* src = x + r * sh.ld + c;
        u32x4 raw; raw.x = 0u; raw.y = 0u; raw.z = 0u; raw.w = 0u;
        if (valid) raw = load16(src);
        uint32_t mg = 0u, mg5 = 0u;
        if (mode == kScaleGam) { const uint32_t* gw = gam_words(gam, group_rows, r); mg = gw[0]; mg5 = gw[1]; }
        sub_block_body<CRIT, DEFER, FAKE>(raw, src, valid, l, r * cpr + cb, o, FAKE ? nullptr : o.fp8 + r * o.ld_fp8 + c,
                                          o.bf16 ? o.bf16 + r * o.ld_bf16 + c : nullptr, FAKE ? o.fake + r * o.ld_fake + c : nullptr,
                                          th, mode, mg, mg5, three != 0u);
    }
}

// ======================================================================================
// Per-tensor granularity (Section 4.1.1 "Per-Tensor"): pass A = global amax, pass B = quantize
// with the global scale, pass C = sums of the per-workgroup error partials in binary64, the decision,
// and the copy of a BF16 fallback that pass B has not already written.
// Everything is stream-ordered; the host never waits.
// ======================================================================================
constexpr int kTensorChunksPerThread = 8;                       // 16-byte chunks per thread in pass B
constexpr int kTensorChunksPerBlock = 256 * kTensorChunksPerThread;
constexpr int kSmallChunksPerThread = 2;                        // ... in pass A of a small operand with padded rows that is alone (see one_max_chunks)
constexpr int kAmaxOneTile = 768;        // tiles of a pass-A launch up to which every one gets a workgroup (three per compute unit); also the size of
                                         // the partials' arrays.  1251 tiles of padded rows: 50.8 us per call at 512 workgroups, 51.9 at 1251
constexpr int kMaxAmaxBlocks = 512;      // pass A of larger launches, all its workgroups resident.  The two parts of the six gradients of
                                         // a layer (256 and 224 MiB) take 45 + 39 us at 512, 49 + 39 us at 2048 with three resident per
                                         // compute unit; the whole layer 409 us at 512, 411 at 384, 413 at 768, 428 at 2048
constexpr int kProveMaxWg = 8192;      // workgroups of one launch (and partial records per operand) of the block-shaped GAM pre-pass

__device__ __forceinline__ uint32_t block_allmax_u32(uint32_t v, uint32_t* sh4) {
    const uint32_t wv = wave_allmax_u32(v);
    if ((threadIdx.x & 63) == 0) sh4[threadIdx.x >> 6] = wv;
    __syncthreads();
    const uint32_t r = max(max(sh4[0], sh4[1]), max(sh4[2], sh4[3]));
    __syncthreads();
    return r;
}
__device__ __forceinline__ uint32_t amax2_of(const u32x4& v, uint32_t a2) {
#pragma unroll
    for (int j = 0; j < 4; ++j) a2 = pk_max_u16(a2, v[j] & 0x7FFF7FFFu);
    return a2;
}

// A partial word of pass A: low half = amax pattern; high half = (smallest non-zero pattern - 1) when the three-way
// recipe needs it for Eq. (4) (0xFFFF: no non-zero element seen), else 0.
__device__ __forceinline__ uint32_t block_allmin_u16(uint32_t v, uint32_t* sh4) { return 0xFFFFu - block_allmax_u32(0xFFFFu - v, sh4); }

// Operands whose rows are longer than the operand is wide (column slices of a fused buffer, padded rows) go through the same
// tiles as dense ones: 16-byte chunks numbered row by row, a tile is kTensorChunksPerBlock consecutive chunks.  A tile's first
// chunk is divided by the chunks per row once (multiplication by a reciprocal, exact below 2^31), a lane's chunks follow by
// adding 256 and wrapping at the row's end; addresses are 32-bit byte offsets from the tile's first row, used with
// bounds-checked buffer accesses.  An operand whose tiles span 2 GB or more (a few columns of very long rows), or whose chunk
// numbers leave those ranges, is `wide`: plain 64-bit arithmetic, one chunk at a time.
// Bound by HBM like the dense form.  Measured with its 1 x 128 sibling (SubRows) on a pair of 4099 x 5000 column slices of
// 10 000-element rows in one call with statistics: 50.8 us, against 103.5 us with kernels of one 16-byte chunk per lane that
// proved no fallback (a third read of the gradient) and took their statistics in launches of their own.
struct RowMap {
    int64_t ld;                    // elements, of x
    uint32_t cpr;                  // chunks per row (0: wide)
    uint32_t mul, shift;           // reciprocal of cpr, see recip_div
    uint32_t step_r, step_c;       // 256 chunks further: rows and chunks
};
__device__ __forceinline__ uint32_t row_div(const RowMap& m, uint32_t n) { return recip_div(n, m.mul, m.shift); }
struct RowPos {
    uint32_t r, c;                 // row inside the tile, chunk inside the row
};
__device__ __forceinline__ int64_t row_tile_first(const RowMap& m, int64_t c_first, uint32_t tid, RowPos& p) {
    const int64_t row0 = c_first < 0x7FFFFFFF ? (int64_t)row_div(m, (uint32_t)c_first) : c_first / m.cpr;      // uniform over the workgroup
    const uint32_t n = (uint32_t)(c_first - row0 * m.cpr) + tid;
    p.r = row_div(m, n);
    p.c = n - p.r * m.cpr;
    return row0;
}
__device__ __forceinline__ void row_step(const RowMap& m, RowPos& p) {
    p.r += m.step_r;
    p.c += m.step_c;
    const bool wrap = p.c >= m.cpr;
    p.c -= wrap ? m.cpr : 0u;
    p.r += wrap ? 1u : 0u;
}
// Byte offset from the tile's first row of a chunk of CHUNK bytes, rows of `row_bytes` bytes (both factors below 2^24).
template <int CHUNK>
__device__ __forceinline__ uint32_t row_off(const RowPos& p, uint32_t row_bytes, bool live) {
    return off_if(live, __umul24(p.r, row_bytes) + p.c * CHUNK);
}

// Smallest non-zero magnitude pattern of the operand from the partial words (0 when it has no non-zero element).
template <int T>             // lanes of the workgroup
__device__ __forceinline__ uint32_t global_amin_bits(const uint32_t* __restrict__ part, int n_part_amax) {
    __shared__ uint32_t sh[T / 64];
    uint32_t m = 0xFFFFu;
    for (int i = threadIdx.x; i < n_part_amax; i += T) m = min(m, part[i] >> 16);
    m = 0xFFFFu - wave_allmax_u32(0xFFFFu - m);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < T / 64; ++k) m = min(m, sh[k]);
    return m == 0xFFFFu ? 0u : m + 1u;
}
// The E5M2 payload of a whole operand (three-way recipe, per-tensor granularity): one more sweep that overwrites the
// E4M3 codes (or the fake-quantized values) of pass B.  One 8-element chunk:
__device__ __forceinline__ void requant_chunk_e5m2(const uint16_t* __restrict__ src, uint8_t* __restrict__ d8, uint16_t* __restrict__ df,
                                                   float s5, float s_inv, bool fast) {
    if (fast) {
        const u32x4 raw = load16(src);
        float e0 = 0.0f, e1 = 0.0f;
        u32x4 deq;
        if (df) { (void)quant8_fast_deq<true, true>(raw, s5, s_inv, e0, e1, deq); store16(df, deq); }
        else store8(d8, quant8_fast_deq<true, false>(raw, s5, s_inv, e0, e1, deq));
    } else {
        (void)quant8_careful_mem<true>(src, s5, df ? nullptr : d8, df, s_inv);
    }
}

struct TensorPartials {   // one slot per pass-B workgroup (at most kMaxQuantBlocks)
    float* err;
    float* err5;
    uint32_t* zero;        // zero elements seen by the workgroup (padding chunks count as zeros)
};
constexpr int kMaxQuantBlocks = 16384;
constexpr int64_t kMaxTensorTiles = 2000ll * kMaxQuantBlocks;      // of one operand: pass B's zero counters (16 bits per lane, 32 a tile) last 2047
static_assert((kMaxTensorTiles / kMaxAmaxBlocks + 1) * kTensorChunksPerBlock * 8 <= 0xFFFFFFFFll,
              "the flush count of a pass-A workgroup is 32 bits wide");
constexpr int kSoloQuantBlocks = 1280;     // pass B of a per-tensor operand that is alone in its launches: persistent workgroups
constexpr int kQuantOneTile = 1536;        // ... unless its tiles all fit the chip at once (six workgroups per compute unit)

// Same result on every thread, two barriers, fixed summation order.
template <typename T>
__device__ __forceinline__ T block_sum_shfl(T v, T* sh4) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
    if ((threadIdx.x & 63) == 0) sh4[threadIdx.x >> 6] = v;
    __syncthreads();
    const T r = (sh4[0] + sh4[1]) + (sh4[2] + sh4[3]);
    __syncthreads();
    return r;
}

struct TileSums {
    float e0, e1, f0, f1;
};
__device__ __forceinline__ TileSums operator+(const TileSums& a, const TileSums& b) { return {a.e0 + b.e0, a.e1 + b.e1, a.f0 + b.f0, a.f1 + b.f1}; }
struct TensorAcc {
    TileSums s;
    uint32_t zero2;
};
__device__ __forceinline__ uint32_t zero2_of(const u32x4& v, uint32_t z2) {
#pragma unroll
    for (int j = 0; j < 4; ++j) z2 = pk_add_u16(z2, pk_is_zero_u16(v[j] & 0x7FFF7FFFu));
    return z2;
}
template <int CRIT>
__device__ __forceinline__ void tensor_publish(const TensorAcc& a, const TensorPartials& tp, int slot) {
    __shared__ float shf[8];
    __shared__ uint32_t shu[4];
    const float werr = wave_allsum_f32(a.s.e0 + a.s.e1);
    const uint32_t wzero = wave_allsum_u32(fold_add16(a.zero2));
    float werr5 = 0.0f;
    if constexpr (CRIT == kCritEq3) werr5 = wave_allsum_f32(a.s.f0 + a.s.f1);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { shf[w] = werr; shf[4 + w] = werr5; shu[w] = wzero; }
    __syncthreads();
    if (threadIdx.x == 0) {
        tp.err[slot] = (shf[0] + shf[1]) + (shf[2] + shf[3]);
        tp.zero[slot] = (shu[0] + shu[1]) + (shu[2] + shu[3]);
        if constexpr (CRIT == kCritEq3) tp.err5[slot] = (shf[4] + shf[5]) + (shf[6] + shf[7]);
    }
}

// A thread's share of the per-workgroup partial sums of pass B (slots threadIdx.x, threadIdx.x + 256, ... in that order).
// Eight slots' loads are in flight together: the workgroup that does this is on the critical path of the call (one
// dependent load per slot took 11 round trips for the 2731 slots of an operand of the layer sweep).  A slot beyond the
// end adds +0, which leaves the (non-negative) sums as they are, so the result is that of the plain loop bit for bit.
template <int CRIT>
__device__ __forceinline__ void tensor_partial_sums(const float* __restrict__ err, const float* __restrict__ err5,
                                                    const uint32_t* __restrict__ zero, int n_slots, double& se, double& se5,
                                                    unsigned long long& sz) {
    for (int i0 = threadIdx.x; i0 < n_slots; i0 += 8 * 256) {
        float e[8], e5[8];
        uint32_t z[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * 256;
            const bool ok = i < n_slots;
            const int ic = ok ? i : n_slots - 1;           // always a valid slot: the loads need no branch
            const float ev = err[ic];
            const uint32_t zv = zero[ic];
            e[u] = ok ? ev : 0.0f;
            z[u] = ok ? zv : 0u;
            if constexpr (CRIT == kCritEq3) { const float e5v = err5[ic]; e5[u] = ok ? e5v : 0.0f; } else e5[u] = 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            se += (double)e[u];
            sz += z[u];
            if constexpr (CRIT == kCritEq3) se5 += (double)e5[u];
        }
    }
}
// Copies `n_chunks` 16-byte chunks from x to dst with workgroup `b` of `nb`: tiles of 1024 consecutive chunks (16 KB),
// four 16-byte loads in flight per lane.
__device__ __forceinline__ void copy_chunk_tiles(const uint16_t* __restrict__ x, uint16_t* __restrict__ dst, int64_t n_chunks, int b, int nb) {
    const int64_t n_tiles = (n_chunks + 1023) / 1024;
    for (int64_t ct = b; ct < n_tiles; ct += nb) {
        const int64_t c0 = ct * 1024 + threadIdx.x;
        if (c0 + 3 * 256 < n_chunks) {
            u32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = load16(x + (c0 + u * 256) * 8);
#pragma unroll
            for (int u = 0; u < 4; ++u) store16(dst + (c0 + u * 256) * 8, v[u]);
        } else {
            for (int u = 0; u < 4; ++u)
                if (c0 + u * 256 < n_chunks) store16(dst + (c0 + u * 256) * 8, load16(x + (c0 + u * 256) * 8));
        }
    }
}

// ======================================================================================
// De-quantize / de-scale (Section 4, Figure 4).  Blocks whose width is a multiple of 8 (or the whole row): tiles of consecutive
// 16-byte output chunks, several operands in a launch; where rows are too long for the tiles' 32-bit offsets, grid.x =
// 128-column strip, grid.y strides over groups of 16 rows, one chunk per thread and row.  Blocks one column wide: one workgroup
// per 128 x 128 tile, so that a thread's 8 column scales are inverted once per tile.
// ======================================================================================
__device__ __forceinline__ float dequant_scale(const float* __restrict__ scale, const uint8_t* __restrict__ e8m0,
                                               const uint32_t* __restrict__ gmant, int64_t p, uint32_t mk, int64_t band) {
    // stored GAM form (Algorithm 1): the scale is rebuilt from the group's shared mantissa and the block's E8M0 byte
    return e8m0 ? __uint_as_float(((uint32_t)e8m0[p] << 23) | gmant[2 * band + (mk == 2u ? 1 : 0)]) : scale[p];
}
// 1 / s, correctly rounded; a NaN scale gives the default NaN, so that products with it convert as pk_bf16_rne expects (the
// decoded NaN codes are default NaNs too).
__device__ __forceinline__ float dequant_inverse(float s) {
    const float v = 1.0f / s;
    return v != v ? __uint_as_float((__float_as_uint(v) & 0x80000000u) | 0x7FC00000u) : v;
}
template <bool E5M2>
__device__ __forceinline__ u32x4 dequant8(const u32x2& q, float s_inv) {
    u32x4 out;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int word = (int)(j < 2 ? q.x : q.y);
        const f32x2 v = (j & 1) ? cvt_pk_f32<E5M2>(word, true) : cvt_pk_f32<E5M2>(word, false);
        out[j] = pk_bf16_rne(v.x * s_inv, v.y * s_inv);
    }
    return out;
}
// One chunk at a time, any leading dimensions (rows too long for the tiles below).
__global__ __launch_bounds__(256) void k_dequant(StatsGeom g, int pr_log2, int pc_log2, const uint8_t* __restrict__ fp8, int64_t ld_fp8,
                                                 const float* __restrict__ scale, const uint8_t* __restrict__ mask,
                                                 const uint16_t* __restrict__ bf16, int64_t ld_bf16, uint16_t* __restrict__ y,
                                                 int64_t ld_y, const uint8_t* __restrict__ e8m0, const uint32_t* __restrict__ gmant,
                                                 int64_t group_rows) {
    const int64_t c = (int64_t)blockIdx.x * 128 + (threadIdx.x & 15) * 8;
    if (c >= g.cols) return;
    for (int64_t r = (int64_t)blockIdx.y * 16 + (threadIdx.x >> 4); r < g.rows; r += (int64_t)gridDim.y * 16) {
        const int64_t p = (r >> pr_log2) * g.gc + (c >> pc_log2);
        const uint32_t mk = mask[p];
        if (mk == 1u) {
            if (bf16) store16(y + r * ld_y + c, load16(bf16 + r * ld_bf16 + c));
            continue;
        }
        const float s_inv = dequant_inverse(dequant_scale(scale, e8m0, gmant, p, mk, group_rows ? r / group_rows : 0));
        const u32x2 q = *reinterpret_cast<const u32x2*>(fp8 + r * ld_fp8 + c);
        store16(y + r * ld_y + c, mk == 2u ? dequant8<true>(q, s_inv) : dequant8<false>(q, s_inv));
    }
}
// Blocks whose width is a multiple of 8: tiles of 1024 consecutive 16-byte output chunks (see RowMap) of one operand per
// workgroup, four per lane.  Bound by HBM (1 byte read and 2 written per element, 2 and 2 in BF16 blocks), so what counts is that
// no load waits for another one: the masks and scales are loaded together, then the payload chunks (FP8 or BF16 as the mask says;
// the other form's load has no address and moves nothing).  8192 x 14336 at 1x128, a tenth of the blocks in BF16: 60 us =
// 6.1 TB/s, against 93 us with one chunk in flight per lane; eight chunks per lane 63 us (101 registers), two 60 us.  14336 x 4096
// without BF16 blocks: 27.0 us; 30.9 us with non-temporal payload loads (the FP8 bytes may still lie in the Infinity Cache,
// where such loads do not look after them), 28.4 us before.
constexpr int kDeqChunks = 4;
constexpr int kMaxGroupDeq = 16;
struct DeqOp {
    RowMap rm;                      // of y; rm.ld is not used
    int64_t n_chunks, gc;
    int32_t pr_log2, pc_log2;
    const uint8_t* fp8;
    const float* scale; const uint8_t* mask;
    const uint16_t* bf16;
    uint16_t* y;
    const uint8_t* e8m0; const uint32_t* gmant;
    uint32_t ld_fp8, ld_bf16, ld_y;
    uint32_t group_rows, group_mul, group_shift;      // stored GAM form with bands of rows as groups (group_rows = 0: one group)
};
struct GroupDeq {
    int n;
    int32_t tile_end[kMaxGroupDeq];
    DeqOp op[kMaxGroupDeq];
};
__global__ __launch_bounds__(256) void k_dequant_group(GroupDeq gd) {
    constexpr int N = kDeqChunks, kTile = 256 * N;
    const int op = group_find32(gd.tile_end, gd.n, blockIdx.x);
    const DeqOp& t = gd.op[op];
    const int64_t c_first = (int64_t)(blockIdx.x - (op ? gd.tile_end[op - 1] : 0)) * kTile;
    const int64_t left = t.n_chunks - c_first;
    const uint32_t valid = (uint32_t)(left < kTile ? left : kTile);
    RowPos pos0;
    const int64_t row0 = row_tile_first(t.rm, c_first, threadIdx.x, pos0);
    const int64_t br0 = row0 >> t.pr_log2;                                // block row of the tile's first row
    const uint8_t* __restrict__ mask = t.mask + br0 * t.gc;
    const float* __restrict__ scale = t.scale ? t.scale + br0 * t.gc : nullptr;
    const uint8_t* __restrict__ e8m0 = t.e8m0 ? t.e8m0 + br0 * t.gc : nullptr;
    uint32_t mk[N];
    float s[N];
    RowPos pos = pos0;
    uint32_t pp[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const bool live = threadIdx.x + u * 256u < valid;
        const uint32_t br = (uint32_t)(((row0 + pos.r) >> t.pr_log2) - br0);
        pp[u] = live ? br * (uint32_t)t.gc + ((pos.c * 8u) >> t.pc_log2) : 0u;      // (block 0 of the tile exists)
        mk[u] = mask[pp[u]];
        row_step(t.rm, pos);
    }
    if (e8m0) {
        pos = pos0;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const uint64_t row = (uint64_t)row0 + (threadIdx.x + u * 256u < valid ? pos.r : 0u);
            const uint64_t band = t.group_rows ? (row < 0x7FFFFFFFu ? recip_div((uint32_t)row, t.group_mul, t.group_shift) : row / t.group_rows) : 0u;
            s[u] = __uint_as_float(((uint32_t)e8m0[pp[u]] << 23) | t.gmant[2 * band + (mk[u] == 2u ? 1 : 0)]);
            row_step(t.rm, pos);
        }
    } else {
#pragma unroll
        for (int u = 0; u < N; ++u) s[u] = scale[pp[u]];
    }
    const BufRsrc r8 = make_buf(t.fp8 + row0 * t.ld_fp8), ry = make_buf(t.y + row0 * t.ld_y);
    const BufRsrc rb = make_buf_window(t.bf16 + row0 * t.ld_bf16, t.bf16 ? 0x7FFFFFFFu : 0u);
    u32x2 q[N];
    u32x4 keep[N];
    bool some_keep = false, some_e5 = false;
    pos = pos0;
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const bool live = threadIdx.x + u * 256u < valid;
        q[u] = buf_load8(r8, row_off<8>(pos, t.ld_fp8, live && mk[u] != 1u), 0u);
        some_keep |= live && mk[u] == 1u;
        some_e5 |= live && mk[u] == 2u;
        row_step(t.rm, pos);
    }
    if (__any(some_keep)) {
        pos = pos0;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            keep[u] = buf_load16(rb, row_off<16>(pos, t.ld_bf16 * 2u, threadIdx.x + u * 256u < valid && mk[u] == 1u), 0u);
            row_step(t.rm, pos);
        }
    } else {
#pragma unroll
        for (int u = 0; u < N; ++u) keep[u] = u32x4{0u, 0u, 0u, 0u};
    }
    auto emit = [&](auto mixed) {
        pos = pos0;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const float s_inv = dequant_inverse(s[u]);
            u32x4 out = dequant8<false>(q[u], s_inv);
            if constexpr (decltype(mixed)::value) {
                const u32x4 out5 = dequant8<true>(q[u], s_inv);
#pragma unroll
                for (int j = 0; j < 4; ++j) out[j] = mk[u] == 2u ? out5[j] : out[j];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) out[j] = mk[u] == 1u ? keep[u][j] : out[j];
            const bool put = threadIdx.x + u * 256u < valid && (mk[u] != 1u || t.bf16 != nullptr);
            buf_store16(ry, row_off<16>(pos, t.ld_y * 2u, put), out);
            row_step(t.rm, pos);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (__any(some_e5)) emit(std::true_type{});
    else emit(std::false_type{});
}
__global__ __launch_bounds__(256) void k_dequant_columns(StatsGeom g, int pr_log2, const uint8_t* __restrict__ fp8, int64_t ld_fp8,
                                                         const float* __restrict__ scale, const uint8_t* __restrict__ mask,
                                                         const uint16_t* __restrict__ bf16, int64_t ld_bf16, uint16_t* __restrict__ y,
                                                         int64_t ld_y, const uint8_t* __restrict__ e8m0, const uint32_t* __restrict__ gmant,
                                                         int64_t group_rows) {
    const int64_t c = (int64_t)blockIdx.x * 128 + (threadIdx.x & 15) * 8;
    if (c >= g.cols) return;
    for (int64_t tr = blockIdx.y; tr * 128 < g.rows; tr += gridDim.y) {
        const int64_t band = group_rows ? tr * 128 / group_rows : 0;        // (a band holds whole 128 x 1 blocks)
        const int64_t p0 = ((tr * 128) >> pr_log2) * g.gc + c;
        float s_inv[8];
        uint32_t mk[8];
        bool any_bf16 = false;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            mk[j] = mask[p0 + j];
            any_bf16 |= mk[j] == 1u;
            s_inv[j] = 1.0f / dequant_scale(scale, e8m0, gmant, p0 + j, mk[j], band);
        }
#pragma unroll 1
        for (int i = 0; i < 8; ++i) {
            const int64_t r = tr * 128 + (threadIdx.x >> 4) + i * 16;
            if (r >= g.rows) break;
            const u32x2 q = *reinterpret_cast<const u32x2*>(fp8 + r * ld_fp8 + c);
            u32x4 keep; keep.x = 0u; keep.y = 0u; keep.z = 0u; keep.w = 0u;
            if (any_bf16) keep = bf16 ? load16(bf16 + r * ld_bf16 + c) : load16(y + r * ld_y + c);
            u32x4 out;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int word = (int)(j < 2 ? q.x : q.y);
                const f32x2 v4 = (j & 1) ? cvt_pk_f32<false>(word, true) : cvt_pk_f32<false>(word, false);
                const f32x2 v5 = (j & 1) ? cvt_pk_f32<true>(word, true) : cvt_pk_f32<true>(word, false);
                const uint32_t lo = mk[2 * j] == 1u ? (keep[j] & 0xFFFFu) : f32_to_bf16_rne((mk[2 * j] == 2u ? v5.x : v4.x) * s_inv[2 * j]);
                const uint32_t hi = mk[2 * j + 1] == 1u ? (keep[j] >> 16) : f32_to_bf16_rne((mk[2 * j + 1] == 2u ? v5.y : v4.y) * s_inv[2 * j + 1]);
                out[j] = lo | (hi << 16);
            }
            store16(y + r * ld_y + c, out);
        }
    }
}

// ======================================================================================
// Selection statistics (Section 4.1.3)
// ======================================================================================
struct StatsDev {   // must match mor_stats in include/mor.h
    unsigned long long n_part, n_fp8_part, n_bf16_part, n_elem_fp8, n_elem_bf16, nnz_total, n_near_threshold;
    double err_sum_total, mean_err;
    uint32_t hist[12];
    uint32_t reserved;      // flags
    uint32_t reserved2;
    unsigned long long n_e5m2_part, n_elem_e5m2;
};
// Number of elements of block p: blocks at the right / bottom edge of a ragged tensor are smaller.
__device__ __forceinline__ unsigned long long block_elems(const StatsGeom& g, int64_t p) {
    if (g.uniform) return (unsigned long long)(g.pr * g.pc);
    const int64_t br = p / g.gc, bc = p - br * g.gc;
    const int64_t h = g.rows - br * g.pr < g.pr ? g.rows - br * g.pr : g.pr;
    const int64_t w = g.cols - bc * g.pc < g.pc ? g.cols - bc * g.pc : g.pc;
    return (unsigned long long)(h * w);
}
// What a wave has counted: the counters are the same in all its lanes (ballots: no lane-by-lane counters to be summed afterwards), the
// sums are each lane's own until stats_reduce.  These kernels are chains of latencies: with fifteen counters per lane summed over the
// waves twice, a lone 1024 x 4096 operand of 128 x 128 blocks took 10.8 us per call with statistics, 9.3 now (64 x 64 13.7 / 11.6,
// 128 x 1 24.6 / 20.9).
struct StatsTally {
    double e;
    unsigned long long n, eb, e5;        // non-zeros; elements in BF16 blocks; elements in E5M2 blocks
    uint32_t c[kStatCnt];
};
__device__ __forceinline__ void tally_clear(StatsTally& a) {
    a.e = 0.0; a.n = 0ull; a.eb = 0ull; a.e5 = 0ull;
#pragma unroll
    for (int k = 0; k < kStatCnt; ++k) a.c[k] = 0u;
}
// One block per lane; all lanes of the wave call (`ok`: this lane has a block).  `elems()` gives the block's elements.
template <class F>
__device__ __forceinline__ void tally(bool ok, float es, uint32_t nz, uint32_t mk, F elems, float th, float near_tol, StatsTally& a) {
    const float metric = nz ? es / (float)nz : 0.0f;           // binary32, IEEE division
    const float m = metric < __builtin_inff() ? metric : __builtin_inff();                // (NaN counts in the last bin, as in stats_bin)
    uint32_t at_least = (uint32_t)__popcll(__ballot(ok));
#pragma unroll
    for (int k = 1; k <= 11; ++k) {
        const uint32_t v = (uint32_t)__popcll(__ballot(ok && m >= (float)(0.005 * k)));
        a.c[k - 1] += at_least - v;
        at_least = v;
    }
    a.c[11] += at_least;
    a.c[12] += (uint32_t)__popcll(__ballot(ok && mk == 1u));
    a.c[13] += (uint32_t)__popcll(__ballot(ok && fabs((double)metric - (double)th) <= (double)near_tol * (double)th));
    a.c[14] += (uint32_t)__popcll(__ballot(ok && mk == 2u));
    if (ok) {
        a.e += (double)es;
        a.n += nz;
        if (mk == 1u) a.eb += elems();
        if (mk == 2u) a.e5 += elems();
    }
}
// `n` blocks from p0 on, step `stride` (a multiple of 64) per round of the workgroup's lanes; four blocks' loads in flight per lane.
__device__ __forceinline__ void tally_blocks(const float* __restrict__ err_sum, const uint32_t* __restrict__ nnz, const uint8_t* __restrict__ mask,
                                             int64_t first, int64_t stride, int64_t n_part, const StatsGeom& geom, float th, float near_tol, StatsTally& a) {
    const int lane = threadIdx.x & 63;
    for (int64_t base = first + (threadIdx.x - lane); base < n_part; base += 4 * stride) {      // uniform over the wave
        float es[4]; uint32_t nz[4], mk[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t p = base + lane + u * stride, pc = p < n_part ? p : n_part - 1;        // always a valid block: the loads need no branch
            es[u] = err_sum[pc]; nz[u] = nnz[pc]; mk[u] = mask[pc];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (base + u * stride >= n_part) break;            // uniform over the wave
            const int64_t p = base + lane + u * stride;
            tally(p < n_part, es[u], nz[u], mk[u], [&] { return block_elems(geom, p); }, th, near_tol, a);
        }
    }
}
template <int WAVES>
struct StatsLds {
    uint32_t c[WAVES][16];
    double e[WAVES];
    unsigned long long n[WAVES], eb[WAVES], e5[WAVES];
};
// Sums over the workgroup (one barrier, fixed order): the totals arrive in wave 0's lanes, counter k in lane k's `mine`.
template <int WAVES>
__device__ __forceinline__ void stats_reduce(StatsTally& a, uint32_t& mine, StatsLds<WAVES>& sh) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    a.e = wave_allsum_f64(a.e); a.n = wave_allsum_u64(a.n);
    const bool kept = (a.c[12] | a.c[14]) != 0u;               // uniform over the wave
    if (kept) { a.eb = wave_allsum_u64(a.eb); a.e5 = wave_allsum_u64(a.e5); }
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < kStatCnt; ++k) sh.c[w][k] = a.c[k];
        sh.e[w] = a.e; sh.n[w] = a.n; sh.eb[w] = a.eb; sh.e5[w] = a.e5;
    }
    __syncthreads();
    mine = 0u;
    a.e = 0.0; a.n = 0ull; a.eb = 0ull; a.e5 = 0ull;
    if (w != 0) return;
#pragma unroll
    for (int k = 0; k < WAVES; ++k) {
        mine += sh.c[k][lane < kStatCnt ? lane : 0];
        a.e += sh.e[k]; a.n += sh.n[k]; a.eb += sh.eb[k]; a.e5 += sh.e5[k];
    }
}
__device__ __forceinline__ void stats_finish(StatsDev* st, int64_t n_part, unsigned long long total_elems, double e,
                                             unsigned long long n, unsigned long long n_bf16, unsigned long long n_near,
                                             unsigned long long n_e5, unsigned long long eb, unsigned long long ee5, uint32_t flags) {
    st->n_part = (unsigned long long)n_part;
    st->n_fp8_part = (unsigned long long)n_part - n_bf16 - n_e5;
    st->n_bf16_part = n_bf16;
    st->n_e5m2_part = n_e5;
    st->n_elem_fp8 = total_elems - eb - ee5;
    st->n_elem_bf16 = eb;
    st->n_elem_e5m2 = ee5;
    st->nnz_total = n;
    st->n_near_threshold = n_near;
    st->err_sum_total = e;
    st->mean_err = n ? e / (double)n : 0.0;
    st->reserved = flags;
    st->reserved2 = 0u;
}
// Counter `k` of the totals that stats_reduce has left in wave 0.
__device__ __forceinline__ uint32_t stats_counter(uint32_t mine, int k) { return (uint32_t)__builtin_amdgcn_readlane((int)mine, k); }
// Wave 0 writes the final statistics.
__device__ __forceinline__ void stats_write(StatsDev* out, int64_t n_part, unsigned long long total_elems, const StatsTally& t, uint32_t mine) {
    if (threadIdx.x >= 64) return;
    if (threadIdx.x < 12) out->hist[threadIdx.x] = mine;
    const uint32_t bf16 = stats_counter(mine, 12), near = stats_counter(mine, 13), e5m2 = stats_counter(mine, 14);
    if (threadIdx.x == 0) stats_finish(out, n_part, total_elems, t.e, t.n, bf16, near, e5m2, t.eb, t.e5, 0u);
}

// Up to a few thousand blocks: one workgroup, no atomics on global memory, deterministic sums.
__global__ __launch_bounds__(256) void k_stats_single(int64_t n_part, StatsGeom geom,
                                                      const float* __restrict__ err_sum, const uint32_t* __restrict__ nnz,
                                                      const uint8_t* __restrict__ mask, float th, float near_tol,
                                                      StatsDev* __restrict__ st) {
    __shared__ StatsLds<4> sh;
    StatsTally a;
    uint32_t mine;
    tally_clear(a);
    tally_blocks(err_sum, nnz, mask, 0, 256, n_part, geom, th, near_tol, a);
    stats_reduce(a, mine, sh);
    stats_write(st, n_part, (unsigned long long)(geom.rows * geom.cols), a, mine);
}

// Many blocks: the accumulators live in the output struct, cleared by a tiny kernel first and
// turned into the derived fields by a tiny kernel afterwards (no device-wide fences needed).
__global__ void k_stats_zero(StatsDev* st) {
    if (threadIdx.x < sizeof(StatsDev) / 4) reinterpret_cast<uint32_t*>(st)[threadIdx.x] = 0u;
}
__global__ __launch_bounds__(256) void k_stats_multi(int64_t n_part, StatsGeom geom,
                                                     const float* __restrict__ err_sum, const uint32_t* __restrict__ nnz,
                                                     const uint8_t* __restrict__ mask, float th, float near_tol,
                                                     StatsDev* __restrict__ st) {
    __shared__ StatsLds<4> sh;
    StatsTally a;
    uint32_t mine;
    tally_clear(a);
    tally_blocks(err_sum, nnz, mask, (int64_t)blockIdx.x * 256, (int64_t)gridDim.x * 256, n_part, geom, th, near_tol, a);
    stats_reduce(a, mine, sh);
    if (threadIdx.x >= 64) return;
    if (threadIdx.x < 12 && mine) atomicAdd(&st->hist[threadIdx.x], mine);
    const uint32_t bf16 = stats_counter(mine, 12), near = stats_counter(mine, 13), e5m2 = stats_counter(mine, 14);
    if (threadIdx.x == 0) {
        atomicAdd(&st->err_sum_total, a.e);
        atomicAdd(&st->nnz_total, a.n);
        atomicAdd(&st->n_bf16_part, (unsigned long long)bf16);
        atomicAdd(&st->n_near_threshold, (unsigned long long)near);
        atomicAdd(&st->n_e5m2_part, (unsigned long long)e5m2);
        atomicAdd(&st->n_elem_bf16, a.eb);
        atomicAdd(&st->n_elem_e5m2, a.e5);
    }
}
// Derived fields once every workgroup of k_stats_multi has finished (next kernel on the stream).
__global__ void k_stats_finish(int64_t n_part, unsigned long long total_elems, StatsDev* __restrict__ st) {
    if (threadIdx.x == 0)
        stats_finish(st, n_part, total_elems, st->err_sum_total, st->nnz_total, st->n_bf16_part, st->n_near_threshold,
                     st->n_e5m2_part, st->n_elem_bf16, st->n_elem_e5m2, 0u);
}

// Running histogram of a tensor's error over training steps (Section 4.1.3): one count per step in the
// bin of (float)mean_err, cleared first on every reset step.
__global__ void k_histogram_update(uint32_t* __restrict__ hist, const StatsDev* __restrict__ st, int clear) {
    const int bin = stats_bin((float)st->mean_err);
    if (threadIdx.x < 12) {
        const uint32_t old = clear ? 0u : hist[threadIdx.x];
        hist[threadIdx.x] = old + ((int)threadIdx.x == bin ? 1u : 0u);
    }
}

// ======================================================================================
// Grouped kernels: one launch processes up to kMaxGroup dense operands of the same granularity and
// criterion.  A training step quantizes many operands (four linear layers x {activation, weight,
// gradient} per transformer block, Section 4), each worth only tens of microseconds of HBM time, so
// per-launch overhead is paid once per group instead of once per operand.  The descriptor tables
// travel in the kernel-argument segment: no staging copy, nothing allocated.
// ======================================================================================
constexpr int kMaxGroup = 8;           // per-tensor operands / GAM pre-pass per launch (their table shares the 4 KB
                                       // kernel-argument segment with the statistics riders)

template <int CRIT, bool FAKE, bool ROWS>
__global__ __launch_bounds__(256) void k_sub1x128_group(GroupSub g) {
    sub_group_body<CRIT, FAKE, false, ROWS>(g, (int64_t)blockIdx.x, (int64_t)gridDim.x, nullptr, 0.0f);
}

// Statistics of sub-tensor operands of a group: pass 1 writes one partial record per workgroup into
// the workspace, pass 2 (one workgroup per operand) combines them in a fixed order.
struct StatsRec {      // 128 bytes
    double e;
    unsigned long long n, eb, e5;
    uint32_t cnt[kStatCnt];
    uint32_t pad[9];
};
struct StatsOp {
    const float* err_sum; const uint32_t* nnz; const uint8_t* mask;
    int64_t n_part;
    StatsGeom geom;
    float th;
    StatsRec* rec;          // [n_wg]
    StatsDev* out;
};
constexpr int kMaxGroupStats = 12;
struct GroupStats {
    int n;
    int32_t wg_end[kMaxGroupStats];
    float near_tol;
    StatsOp op[kMaxGroupStats];
};
// Wave 0 leaves the workgroup's record.
__device__ __forceinline__ void stats_record(StatsRec* r, const StatsTally& t, uint32_t mine) {
    if (threadIdx.x < kStatCnt) r->cnt[threadIdx.x] = mine;
    if (threadIdx.x == 0) { r->e = t.e; r->n = t.n; r->eb = t.eb; r->e5 = t.e5; }
}
// Workgroup of T lanes: its share of an operand's blocks, into its record, or (the operand's only workgroup) the final statistics.
template <int T>
__device__ __forceinline__ void stats_partial_body(const GroupStats& g, int block) {
    __shared__ StatsLds<T / 64> sh;
    const int op = group_find32(g.wg_end, g.n, block);
    const StatsOp& t = g.op[op];
    const int b = block - (op ? g.wg_end[op - 1] : 0);
    const int nb = g.wg_end[op] - (op ? g.wg_end[op - 1] : 0);
    StatsTally a;
    uint32_t mine;
    tally_clear(a);
    tally_blocks(t.err_sum, t.nnz, t.mask, (int64_t)b * T, (int64_t)nb * T, t.n_part, t.geom, t.th, g.near_tol, a);
    stats_reduce(a, mine, sh);
    if (nb == 1) stats_write(t.out, t.n_part, (unsigned long long)(t.geom.rows * t.geom.cols), a, mine);
    else stats_record(t.rec + b, a, mine);
}
// Sums of up to 256 records by a workgroup of 256 lanes.  Sixteen neighbouring lanes read a record together, eight bytes each (one line
// per record; a record per lane would be a line per lane and load), and what is left of every quadword goes through shared memory.
// Every thread may read the sums from `all` afterwards: the sum, three 64-bit counts, then pairs of counters.
struct RecordSums {
    unsigned long long part[16][16], all[16];
};
__device__ __forceinline__ unsigned long long row_allsum_u64(unsigned long long v) {
    v += dpp_u64<kDppXor1>(v); v += dpp_u64<kDppXor2>(v); v += dpp_u64<kDppHalfMirror>(v); v += dpp_u64<kDppMirror>(v);
    return v;
}
__device__ __forceinline__ double row_allsum_f64(double v) {
    auto sh = [](double x, auto ctrl) { return __longlong_as_double((long long)dpp_u64<decltype(ctrl)::value>((unsigned long long)__double_as_longlong(x))); };
    v += sh(v, std::integral_constant<int, kDppXor1>{}); v += sh(v, std::integral_constant<int, kDppXor2>{});
    v += sh(v, std::integral_constant<int, kDppHalfMirror>{}); v += sh(v, std::integral_constant<int, kDppMirror>{});
    return v;
}
__device__ __forceinline__ void sum_records(const StatsRec* __restrict__ rec, int n_rec, RecordSums& sh) {
    const int tid = threadIdx.x, grp = tid >> 4, k = tid & 15;
    const bool is_sum = k == 0;                                // (an error sum may be infinite: its bits are added as a double, never as integers)
    unsigned long long n = 0ull;                               // a 64-bit count, or two counters side by side (no operand has 2^32 blocks)
    double e = 0.0;
    for (int i0 = grp; i0 < n_rec; i0 += 4 * 16) {
        unsigned long long v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = reinterpret_cast<const unsigned long long*>(rec + (i0 + u * 16 < n_rec ? i0 + u * 16 : i0))[k];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool ok = i0 + u * 16 < n_rec;
            n += ok ? v[u] : 0ull;
            e += ok && is_sum ? __longlong_as_double((long long)v[u]) : 0.0;
        }
    }
    sh.part[grp][k] = is_sum ? (unsigned long long)__double_as_longlong(e) : n;
    __syncthreads();
    const unsigned long long v = sh.part[k][grp];              // sixteen lanes per quadword now
    const unsigned long long c = row_allsum_u64(v);
    const double f = row_allsum_f64(grp == 0 ? __longlong_as_double((long long)v) : 0.0);
    if (k == 0) sh.all[grp] = grp == 0 ? (unsigned long long)__double_as_longlong(f) : c;
    __syncthreads();
}
__device__ __forceinline__ uint32_t record_counter(const RecordSums& sh, int k) { return (uint32_t)(sh.all[4 + (k >> 1)] >> (32 * (k & 1))); }
__device__ __forceinline__ void stats_final_body(const GroupStats& g, int op) {
    __shared__ RecordSums sh;
    const StatsOp& t = g.op[op];
    const int nb = g.wg_end[op] - (op ? g.wg_end[op - 1] : 0);       // <= kStatsMaxWg = 256
    if (nb == 1) return;                                             // already final
    sum_records(t.rec, nb, sh);
    if (threadIdx.x < 12) t.out->hist[threadIdx.x] = record_counter(sh, threadIdx.x);
    if (threadIdx.x == 0)
        stats_finish(t.out, t.n_part, (unsigned long long)(t.geom.rows * t.geom.cols), __longlong_as_double((long long)sh.all[0]), sh.all[1], record_counter(sh, 12),
                     record_counter(sh, 13), record_counter(sh, 14), sh.all[2], sh.all[3], 0u);
}

// ---- statistics launches of their own (operands that found no per-tensor launch to ride on, e.g. a single sub-tensor
//      operand): here the statistics are on the critical path of the call, so the kernels are built for latency --
//      workgroups of 1024 lanes, every lane's loads in flight together, counters by ballots, one barrier.  An operand of up to
//      kStatsDirectParts blocks is finished by one workgroup in one launch; larger ones leave one record per workgroup for
//      the combine launch.
constexpr int kStatsFastThreads = 1024;
constexpr int kStatsFastPerLane = 4;                   // blocks per lane of a partial workgroup
constexpr int64_t kStatsDirectParts = 16384;           // one workgroup, 16 blocks per lane at most
__global__ __launch_bounds__(kStatsFastThreads) void k_stats_group_partial(GroupStats g) { stats_partial_body<kStatsFastThreads>(g, (int)blockIdx.x); }
// Combine launch: one workgroup per operand.
__global__ __launch_bounds__(256) void k_stats_group_final(GroupStats g) { stats_final_body(g, (int)blockIdx.x); }

// ======================================================================================
// Tensor-level decision over sub-tensor scaling (Section 3.1): the deferred block kernels wrote
// err_sum / nnz per block; aggregate sum(err_sum) / sum(nnz), decide once, broadcast the mask.
// ======================================================================================
// Grouped: every operand with a tensor-level decision shares two launches -- partial sums per workgroup, then the decision
// (re-derived by every workgroup of the operand from the partials in a fixed order, so all agree) with the mask
// broadcast and the conditional copy of the BF16 fallback.
constexpr int kScopeBlocks = 256;       // partial records per operand
constexpr int kMaxGroupScope = 16;
struct ScopeOp {
    const float* err_sum; const float* err5_sum; const uint32_t* nnz; uint8_t* mask;
    int64_t n_part;
    double* part_err; double* part_err5; unsigned long long* part_nnz;     // [kScopeBlocks] each
    uint32_t* decision;                                                    // [1]
    const uint32_t* proven;                                                // non-null and [0] != 0: the block kernel wrote the fallback
    float th;
    int32_t crit;
    int32_t n_red;                                                         // workgroups of the reduce pass (<= kScopeBlocks)
    // fallback copy
    const uint16_t* x; uint16_t* bf16;
    int64_t rows, cols, ld, ld_bf16;
    // per-channel columns: the blocks' sums are still those of the strips, [n_strips x cols_padded]; the reduce pass adds them up
    ColumnSums col;
    // selection statistics: all blocks get one decision, so the reduce pass can count everything that does not depend on it
    StatsDev* stats;                                                       // optional
    StatsRec* rec;                                                         // [n_red]
    float near_tol;
};
struct GroupScope {
    int n;
    int32_t red_end[kMaxGroupScope], copy_end[kMaxGroupScope];
    ScopeOp op[kMaxGroupScope];
};
// Error sums and non-zero count of a column from those of its strips (binary64, fixed order), into the outputs: what the combine launch of
// the per-channel columns does where the columns decide one by one.  (The third load of a strip is always made, from the E4M3 sums where
// there are no others: a branch around it leaves one load in flight, and a loop for each criterion makes the kernel so long that small
// operands of other granularities pay for it.  us per call, Eq. 3 8192 x 4096 59.2 with the branch, 50.1 with two loops, 49.9 like this;
// 128 x 128 blocks 1024 x 4096 11.3, 11.5, 11.3.)
__device__ __forceinline__ void column_sums(const ScopeOp& t, int64_t c, bool live, bool eq3, float& es, uint32_t& nz, float& es5) {
    double e = 0.0, e5 = 0.0;
    unsigned long long z = 0ull;
    const float* __restrict__ err5 = eq3 ? t.col.err5 : t.col.err;
    for (int s0 = 0; s0 < t.col.n_strips; s0 += 8) {
        float ev[8], e5v[8];
        uint32_t zv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int64_t at = (int64_t)(s0 + k < t.col.n_strips ? s0 + k : s0) * t.col.cols_padded + c;      // always a valid strip: the loads need no branch
            ev[k] = t.col.err[at]; zv[k] = t.col.zero[at]; e5v[k] = err5[at];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const bool ok = s0 + k < t.col.n_strips;
            e += ok ? (double)ev[k] : 0.0; e5 += ok ? (double)e5v[k] : 0.0; z += ok ? zv[k] : 0u;
        }
    }
    const unsigned long long n = (unsigned long long)((t.rows + 127) / 128) * 128ull - z;      // (rows beyond the tensor were counted as zeros)
    if (__float_as_uint(t.col.amax[c]) >> 16 >= kInfBits) { e = (double)__builtin_inff(); e5 = e; }
    es = (float)e; es5 = (float)e5;
    nz = n > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)n;
    if (!live) return;
    const_cast<float*>(t.err_sum)[c] = es;
    const_cast<uint32_t*>(t.nnz)[c] = nz;
    if (eq3) const_cast<float*>(t.err5_sum)[c] = es5;
}
// Four blocks' loads in flight per lane.  With statistics the same sweep also fills the workgroup's record (histogram bins,
// near-threshold blocks), so no statistics launch follows.
__global__ __launch_bounds__(256) void k_scope_reduce_group(GroupScope g) {
    __shared__ double shd[4];
    __shared__ StatsLds<4> sh;
    const int op = group_find32(g.red_end, g.n, blockIdx.x);
    const ScopeOp& t = g.op[op];
    const int b = blockIdx.x - (op ? g.red_end[op - 1] : 0);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const bool eq3 = t.crit == kCritEq3, want = t.stats != nullptr;
    double e5 = 0.0;
    StatsTally a;
    tally_clear(a);
    const int64_t stride = (int64_t)t.n_red * 256;
    for (int64_t base = (int64_t)b * 256 + w * 64; base < t.n_part; base += 4 * stride) {       // uniform over the wave
        float es[4], es5[4];
        uint32_t nz[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t p = base + lane + u * stride, pc = p < t.n_part ? p : t.n_part - 1;    // always a valid block: the loads need no branch
            if (t.col.n_strips) {                              // uniform over the workgroup
                if (base + u * stride >= t.n_part) break;
                column_sums(t, pc, p < t.n_part, eq3, es[u], nz[u], es5[u]);
            } else { es[u] = t.err_sum[pc]; nz[u] = t.nnz[pc]; es5[u] = eq3 ? t.err5_sum[pc] : 0.0f; }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (base + u * stride >= t.n_part) break;          // uniform over the wave
            const bool ok = base + lane + u * stride < t.n_part;
            e5 += ok ? (double)es5[u] : 0.0;
            if (want) tally(ok, es[u], nz[u], 0u, [] { return 0ull; }, t.th, t.near_tol, a);
            else if (ok) { a.e += (double)es[u]; a.n += nz[u]; }
        }
    }
    if (eq3) { e5 = wave_allsum_f64(e5); if (lane == 0) shd[w] = e5; }
    uint32_t mine;
    stats_reduce(a, mine, sh);                                 // (its barrier also covers shd)
    if (threadIdx.x == 0) { t.part_err[b] = a.e; t.part_nnz[b] = a.n; t.part_err5[b] = eq3 ? (shd[0] + shd[1]) + (shd[2] + shd[3]) : 0.0; }
    if (want) stats_record(t.rec + b, a, mine);
}
// Same decision in every wave that calls it (fixed summation order over the operand's partial records), no barrier.
__device__ __forceinline__ uint32_t scope_decision(const ScopeOp& t) {
    const int lane = threadIdx.x & 63;
    double e = 0.0, e5 = 0.0;
    unsigned long long n = 0;
#pragma unroll
    for (int k = 0; k < kScopeBlocks / 64; ++k) {
        const bool ok = lane + 64 * k < t.n_red;
        const int i = ok ? lane + 64 * k : 0;
        const double ev = t.part_err[i], e5v = t.part_err5[i];
        const unsigned long long nv = t.part_nnz[i];
        e += ok ? ev : 0.0; e5 += ok ? e5v : 0.0; n += ok ? nv : 0ull;
    }
    e = wave_allsum_f64(e);
    if (t.crit == kCritEq3) return (e < wave_allsum_f64(e5)) ? 0u : 1u;
    n = wave_allsum_u64(n);
    return ((n ? e / (double)n : 0.0) < (double)t.th) ? 0u : 1u;
}
__device__ __forceinline__ void scope_copy(const ScopeOp& t, int b, int nb) {
    if (t.ld == t.cols && t.ld_bf16 == t.cols) {
        copy_chunk_tiles(t.x, t.bf16, t.rows * t.cols / 8, b, nb);
    } else {
        const int64_t cpr = t.cols / 8;
        for (int64_t r = b; r < t.rows; r += nb)
            for (int64_t c = threadIdx.x; c < cpr; c += 256) store16(t.bf16 + r * t.ld_bf16 + c * 8, load16(t.x + r * t.ld + c * 8));
    }
}
// Decision (every workgroup re-derives it from the partial records: the same value everywhere), mask broadcast over the
// operand's workgroups, statistics by its first one, then the copy of a BF16 tensor that no earlier pass has proven and written.
__global__ __launch_bounds__(256) void k_scope_copy_group(GroupScope g) {
    __shared__ RecordSums sh;
    const int op = group_find32(g.copy_end, g.n, blockIdx.x);
    const ScopeOp& t = g.op[op];
    const int b = blockIdx.x - (op ? g.copy_end[op - 1] : 0);
    const int nb = g.copy_end[op] - (op ? g.copy_end[op - 1] : 0);
    const uint32_t m = scope_decision(t);
    if (b == 0 && threadIdx.x == 0) t.decision[0] = m;
    for (int64_t p = (int64_t)b * 256 + threadIdx.x; p < t.n_part; p += (int64_t)nb * 256) t.mask[p] = (uint8_t)m;
    if (b == 0 && t.stats) {                                   // uniform over the workgroup
        sum_records(t.rec, t.n_red, sh);
        const unsigned long long total = (unsigned long long)(t.rows * t.cols);
        if (threadIdx.x < 12) t.stats->hist[threadIdx.x] = record_counter(sh, threadIdx.x);
        if (threadIdx.x == 0)
            stats_finish(t.stats, t.n_part, total, __longlong_as_double((long long)sh.all[0]), sh.all[1], m ? (unsigned long long)t.n_part : 0ull,
                         record_counter(sh, 13), 0ull, m ? total : 0ull, 0ull, 0u);
    }
    if (t.bf16 == nullptr || m == 0u || (t.proven && t.proven[0] != 0u)) return;
    scope_copy(t, b, nb);
}
// Operands of few blocks: the decision from the blocks' sums in every workgroup, without the reduce launch before it.  What is read for it lies
// in the L2 cache; a proven operand's workgroups that have no part of the mask to write leave at once.
// A launch is what bounds a small operand here.  us per call, weights with FP32 scales, two launches / this one: 128 x 128 blocks of 256 x 1024 13.6 / 9.2,
// 1 x 128 of 256 x 1024 (2048 blocks) 13.7 / 9.4, 64 x 64 of 4096 x 4096 (4096) 20.7 / 18.8, 1 x 128 of 1024 x 1024 (8192) 13.8 / 12.3 but channels of
// 8192 x 4096 (8192) 27.6 / 27.8; with GAM scales 21.0 / 17.1, 21.3 / 17.4, 27.2 / 25.6, 21.7 / 18.4, 38.1 / 38.3.  With statistics, which one workgroup
// counts: 13.6 / 9.4, 13.5 / 12.4, 22.7 / 25.1, 14.3 / 24.1, 29.7 / 39.8.
constexpr int64_t kScopeDirect = 4096, kScopeDirectStats = 2048;      // blocks of an operand, without and with statistics
__global__ __launch_bounds__(256) void k_scope_direct_group(GroupScope g) {
    __shared__ double she[4], she5[4];
    __shared__ unsigned long long shn[4];
    __shared__ StatsLds<4> sh;
    const int op = group_find32(g.copy_end, g.n, blockIdx.x);
    const ScopeOp& t = g.op[op];
    const int b = blockIdx.x - (op ? g.copy_end[op - 1] : 0);
    const int nb = g.copy_end[op] - (op ? g.copy_end[op - 1] : 0);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, n_part = (int)t.n_part;
    const bool eq3 = t.crit == kCritEq3, copied = t.bf16 == nullptr || (t.proven && t.proven[0] != 0u);
    if (copied && (int64_t)b * 256 >= t.n_part) return;        // (uniform over the workgroup)
    double e = 0.0, e5 = 0.0;
    unsigned long long n = 0ull;
    for (int i0 = tid; i0 < n_part; i0 += 8 * 256) {
        float ev[8], e5v[8];
        uint32_t nv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * 256 < n_part ? i0 + u * 256 : i0;      // always a valid block: the loads need no branch
            ev[u] = t.err_sum[i]; nv[u] = t.nnz[i]; e5v[u] = eq3 ? t.err5_sum[i] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool ok = i0 + u * 256 < n_part;
            e += ok ? (double)ev[u] : 0.0; e5 += ok ? (double)e5v[u] : 0.0; n += ok ? nv[u] : 0u;
        }
    }
    e = wave_allsum_f64(e);
    n = wave_allsum_u64(n);
    if (eq3) e5 = wave_allsum_f64(e5);
    if (lane == 0) { she[w] = e; she5[w] = e5; shn[w] = n; }
    __syncthreads();
    e = (she[0] + she[1]) + (she[2] + she[3]);
    n = (shn[0] + shn[1]) + (shn[2] + shn[3]);
    uint32_t m;
    if (eq3) m = e < (she5[0] + she5[1]) + (she5[2] + she5[3]) ? 0u : 1u;
    else m = ((n ? e / (double)n : 0.0) < (double)t.th) ? 0u : 1u;
    if (b == 0 && tid == 0) t.decision[0] = m;
    for (int p = b * 256 + tid; p < n_part; p += nb * 256) t.mask[p] = (uint8_t)m;
    if (b == 0 && t.stats) {                                   // uniform over the workgroup
        StatsTally a;
        tally_clear(a);
        for (int base = w * 64; base < n_part; base += 4 * 256) {       // uniform over the wave
            float es[4];
            uint32_t nz[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = base + lane + u * 256 < n_part ? base + lane + u * 256 : n_part - 1;
                es[u] = t.err_sum[i]; nz[u] = t.nnz[i];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (base + u * 256 >= n_part) break;           // uniform over the wave
                tally(base + lane + u * 256 < n_part, es[u], nz[u], 0u, [] { return 0ull; }, t.th, t.near_tol, a);
            }
        }
        uint32_t mine;
        stats_reduce(a, mine, sh);
        const unsigned long long total = (unsigned long long)(t.rows * t.cols);
        if (tid < 12) t.stats->hist[tid] = mine;
        if (tid < 64) {
            const uint32_t near = stats_counter(mine, 13);
            if (tid == 0) stats_finish(t.stats, t.n_part, total, a.e, a.n, m ? (unsigned long long)n_part : 0ull, near, 0ull, m ? total : 0ull, 0ull, 0u);
        }
    }
    if (!copied && m != 0u) scope_copy(t, b, nb);
}

// ---- a lone dense 1 x 128 operand: the block kernel gathers the statistics of its workgroups itself (one record per
//      workgroup), so that the call needs one small combine launch afterwards instead of two statistics launches that
//      read the per-block outputs again.  (Combining the records inside the block kernel as well -- the workgroup that
//      draws the last of a set of ticket counters reads all records -- was built and measured: device-wide atomics on one
//      address complete about 15 ns apart, a device-wide release fence per workgroup writes back what its XCD still
//      holds of the payload (80 us per call), and with write-through record stores and two levels of counters the chain
//      of dependent device-scope round trips at the end of the kernel took as long as the launch it was to save.)
constexpr int kSoloRecWords = 20;          // dwords of a workgroup's record in use: 15 counters, pad, the sum (2), non-zeros, pad
struct SoloStats {
    StatsRec* rec;         // [gridDim.x]: 128 bytes apart, the first kSoloRecWords dwords used
    StatsDev* out;
    int64_t n_part;
    unsigned long long total_elems;
    uint32_t edge_missing;     // elements that a block of the last column lacks (ragged operands)
    float near_tol;
    int n_rec;
};
// (Six workgroups per compute unit as for the kernel without statistics: the second launch bound makes the compiler fit
// Eq. 2's variants into 80 registers, which it does without spilling; Eq. 3's variants need more either way.)
template <int CRIT, bool FAKE, bool ROWS, class G>
__device__ __forceinline__ void sub_solo_body(const G& g, StatsRec* rec, float near_tol, int block, int n_blocks, SubStatsShared& ssh) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (threadIdx.x < 17) reinterpret_cast<uint32_t*>(&ssh)[threadIdx.x] = 0u;      // c[16], n
    ssh.e_lane[threadIdx.x] = 0.0;
    ssh.n_lane[threadIdx.x] = 0u;
    __syncthreads();
    sub_group_body<CRIT, FAKE, true, ROWS>(g, (int64_t)block, (int64_t)n_blocks, &ssh, near_tol);
    const double e_w = wave_allsum_f64(ssh.e_lane[threadIdx.x]);
    const uint32_t n_w = wave_allsum_u32(ssh.n_lane[threadIdx.x]);
    if (lane == 0) { ssh.e[w] = e_w; atomicAdd(&ssh.n, n_w); }
    __syncthreads();
    if (w != 0) return;
    uint32_t word = 0u;                                   // one dword of the record per lane
    if (lane < kStatCnt) word = ssh.c[lane];
    const double e_wg = (ssh.e[0] + ssh.e[1]) + (ssh.e[2] + ssh.e[3]);
    const unsigned long long e_bits = (unsigned long long)__double_as_longlong(e_wg);
    if (lane == 16) word = (uint32_t)e_bits;
    if (lane == 17) word = (uint32_t)(e_bits >> 32);
    if (lane == 18) word = ssh.n;
    if (lane < kSoloRecWords) reinterpret_cast<uint32_t*>(rec + block)[lane] = word;
}
template <int CRIT, bool FAKE, bool ROWS>
__global__ __launch_bounds__(256, CRIT == kCritEq3 || ROWS ? 4 : 6) void k_sub1x128_solo_stats(SubRiders g, SoloStats s) {
    __shared__ SubStatsShared ssh;
    sub_solo_body<CRIT, FAKE, ROWS>(g, s.rec, s.near_tol, (int)blockIdx.x, (int)gridDim.x, ssh);
}
// Combine launch of the above: one workgroup, the records in a fixed order.  It is pure latency on the critical path of the call, so a
// record is read by ten neighbouring lanes, eight bytes each (one line per record instead of one line per lane and load), and only
// ten values per group of lanes are left to be summed through shared memory: the launch takes 2.0 us at least and 3.4 on average instead of
// 5.0 and 6.3 with a record per lane (calls of 1000 x 4096 and 8192 x 4096 under the profiler), 1000 x 4096 with statistics 8.3 instead of
// 11.3 us per call, 8192 x 4096 26.5 instead of 29.3.
constexpr int kSoloFinalThreads = 1024;
constexpr int kSoloQ = kSoloRecWords / 2;              // quadwords: seven pairs of counters and one counter, the sum, the non-zeros
template <int T>
__device__ __forceinline__ void solo_final_body(const SoloStats& s) {
    constexpr int kGroups = T / 16;
    __shared__ unsigned long long part[kGroups][kSoloQ];
    __shared__ unsigned long long all[kSoloQ];
    const int tid = threadIdx.x, grp = tid >> 4, k = tid & 15;
    const bool is_sum = k == 8;                                // (an error sum may be infinite: its bits are added as a double, never as integers)
    if (k < kSoloQ) {
        unsigned long long n = 0ull;                           // two counters side by side (no operand has 2^32 blocks), or the non-zeros
        double e = 0.0;
        constexpr int kFlight = T < 1024 ? 16 : 4;             // records' loads in flight per lane
        for (int i0 = grp; i0 < s.n_rec; i0 += kFlight * kGroups) {
            unsigned long long v[kFlight];
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                const int i = i0 + u * kGroups < s.n_rec ? i0 + u * kGroups : i0;      // always a valid record: the loads need no branch
                v[u] = reinterpret_cast<const unsigned long long*>(s.rec + i)[k];
            }
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                const bool ok = i0 + u * kGroups < s.n_rec;
                n += ok ? v[u] : 0ull;
                e += ok && is_sum ? __longlong_as_double((long long)v[u]) : 0.0;
            }
        }
        part[grp][k] = is_sum ? (unsigned long long)__double_as_longlong(e) : n;
    }
    __syncthreads();
    if (tid < 16 * kSoloQ) {                                   // sixteen lanes per quadword
        const int q = tid >> 4, j = tid & 15;
        unsigned long long v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = u < kGroups / 16 ? part[j + 16 * (u < kGroups / 16 ? u : 0)][q] : 0ull;
        const unsigned long long n = row_allsum_u64((v[0] + v[1]) + (v[2] + v[3]));
        auto f = [&](int u) { return __longlong_as_double((long long)v[u]); };
        const double e = row_allsum_f64((f(0) + f(1)) + (f(2) + f(3)));
        if (j == 0) all[q] = q == 8 ? (unsigned long long)__double_as_longlong(e) : n;
    }
    __syncthreads();
    auto count = [&](int c) { return (uint32_t)(all[c >> 1] >> (32 * (c & 1))); };
    if (tid < 12) s.out->hist[tid] = count(tid);
    if (tid == 0)                                              // (no E5M2 blocks here: counter 14 holds the BF16 blocks of a ragged last column)
        stats_finish(s.out, s.n_part, s.total_elems, __longlong_as_double((long long)all[8]), all[9],
                     count(12), count(13), 0ull, 128ull * count(12) - (unsigned long long)s.edge_missing * count(14), 0ull, 0u);
}

__global__ __launch_bounds__(kSoloFinalThreads) void k_solo_stats_final(SoloStats s) { solo_final_body<kSoloFinalThreads>(s); }

// Per-tensor operands of a group share three launches (amax, quantize, finish + fallback copy).
enum : uint32_t { kTensorLean = 1u,       // a proven BF16 operand gets no FP8 payload
                  kTensorReport = 2u,    // the statistics say that the decision was proven
                  kTensorDense = 4u };   // rows without padding (kernels that take both kinds)
struct TensorOp {
    const uint16_t* x;
    int64_t n_chunks, n_tiles;
    int64_t chunks_per_row;              // STRIDED kernels
    KOut o;
    float th;
    uint32_t mode;                       // scaling algorithm
    uint32_t three;                      // type list [E4M3, E5M2, BF16]
    uint32_t flags;                      // kTensorLean, kTensorReport, kTensorDense
    int n_amax, n_slots;                 // workgroups this operand gets in pass A / pass B
    uint32_t* amax_part;                 // [n_amax]
    float* err; float* err5; uint32_t* zero;   // [n_slots] each
    uint32_t* abits;                     // [2]: global amax bits; 1 if pass B wrote the fallback
    uint32_t* flush_part;                // [n_amax] lower bounds on the number of elements certain to flush to zero
    unsigned long long flush_need;       // that many certain flushes prove the BF16 decision (0 = proof not attempted)
    StatsDev* stats;                     // optional
    int64_t keep_from;                   // pass A: tiles from this one on are read without the non-temporal hint
    RowMap rm;                           // operands with padded leading dimensions (STRIDED kernels)
};
template <int N>
struct GroupTensorT {
    int n;
    int32_t amax_end[N], slot_end[N], copy_end[N];   // running workgroup totals per pass
    float near_tol;
    TensorOp op[N];
};
using GroupTensor = GroupTensorT<kMaxGroup>;
using OneTensor = GroupTensorT<1>;
// Element offset of 16-byte chunk `c` in a matrix with rows of `ld` elements, any size (paths that are not bound by it).
template <bool STRIDED>
__device__ __forceinline__ int64_t tensor_chunk_off(const TensorOp& t, int64_t c, int64_t ld) {
    if constexpr (!STRIDED) return c * 8;
    const int64_t cpr = t.chunks_per_row, r = c / cpr;
    return r * ld + (c - r * cpr) * 8;
}
// Pass A also gathers a PROOF of the BF16 decision where one exists.  Section 4.1.3 observes that a
// per-tensor scale falls back as soon as ~2.4 % of the values flush to zero; each flushed non-zero
// element contributes exactly 1 to the error sum of Eq. (1)-(2), so "flushed >= th * N" already implies
// "mean relative error >= th".  An element certainly flushes when |x| < amax * 2^-20 (then
// |x * 448/amax| < 2^-11, below half of E4M3's smallest subnormal); with the lane's RUNNING amax in
// place of the final one the test only becomes stricter, so the count is a lower bound.  When the
// bound reaches flush_need, pass B writes the BF16 fallback in the same sweep and the separate copy
// pass (2 more bytes read per element) is skipped.  The outputs are the same either way.
// Workgroups from `stats_first` on do not belong to pass A: they compute the partial statistics records of the batch's
// sub-tensor operands (whose kernels have already run), in the shadow of this bandwidth-bound pass.
// Elements among CH chunks that are certain to flush, `bound2` (both half-words) being the amax or a lower bound of it.
template <int CH>
__device__ __forceinline__ uint32_t certain_flushes(const u32x4 (&v)[CH], uint32_t bound2) {
    // t = bound with 20 taken off the exponent (0 if that underflows); 1 <= m < t  <=>  m-1 < t-1
    const uint32_t t2 = pk_sub_sat_u16(bound2, 0x0A000A00u);
    const uint32_t tm1 = pk_sub_sat_u16(t2, 0x00010001u);
    uint32_t keep2 = 0u;                       // per half-word: elements NOT certain to flush
#pragma unroll
    for (int u = 0; u < CH; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t mm1 = pk_sub_u16(v[u][j] & 0x7FFF7FFFu, 0x00010001u);     // wraps to 0xFFFF for zeros
            keep2 = pk_add_u16(keep2, pk_is_zero_u16(pk_sub_sat_u16(tm1, mm1)));
        }
    return 8u * CH - fold_add16(keep2);
}
template <bool STRIDED, int CH, class G>
__device__ __forceinline__ void tensor_amax_body(const G& g, int block) {
    constexpr int kTile = 256 * CH;
    constexpr bool kSmall = CH != kTensorChunksPerThread;
    __shared__ uint32_t sh4[4];
    const int op = group_find32(g.amax_end, g.n, block);
    const TensorOp& t = g.op[op];
    const int b = block - (op ? g.amax_end[op - 1] : 0);
    const bool prove = t.flush_need != 0ull;
    const bool three = t.three != 0u;
    uint32_t a2 = 0u, flushed = 0u;
    uint32_t mn2 = 0xFFFFFFFFu;                   // three-way recipe: smallest non-zero pattern, minus one, per half-word
    for (int64_t tile = b; tile < t.n_tiles; tile += t.n_amax) {
        const int64_t c0 = tile * kTile + threadIdx.x;
        // Small tiles are taken whole, chunks beyond the operand as zeros: the reduction over the wave below needs all its lanes.
        if ((kSmall || c0 + (CH - 1) * 256 < t.n_chunks) && !(STRIDED && t.rm.cpr == 0u)) {
            u32x4 v[CH];
            if constexpr (STRIDED) {
                RowPos pos;
                const int64_t row0 = row_tile_first(t.rm, tile * kTile, threadIdx.x, pos);
                const BufRsrc rx = make_buf(t.x + row0 * t.rm.ld);
                const uint32_t row_bytes = (uint32_t)t.rm.ld * 2u;
                uint32_t off[CH];
#pragma unroll
                for (int u = 0; u < CH; ++u) { off[u] = row_off<16>(pos, row_bytes, !kSmall || c0 + u * 256 < t.n_chunks); row_step(t.rm, pos); }
                if (tile >= t.keep_from) {
#pragma unroll
                    for (int u = 0; u < CH; ++u) v[u] = buf_load16_first<true>(rx, off[u], 0u);
                } else {
#pragma unroll
                    for (int u = 0; u < CH; ++u) v[u] = buf_load16_first<false>(rx, off[u], 0u);
                }
            } else {
                // (buffer loads: plain loads that differ in the hint only would be merged into one without it)
                const BufRsrc rx = make_buf(t.x + tile * (kTile * 8));
                if (tile >= t.keep_from) {
#pragma unroll
                    for (int u = 0; u < CH; ++u) v[u] = buf_load16_first<true>(rx, threadIdx.x * 16u + u * 4096u, 0u);
                } else {
#pragma unroll
                    for (int u = 0; u < CH; ++u) v[u] = buf_load16_first<false>(rx, threadIdx.x * 16u + u * 4096u, 0u);
                }
            }
#pragma unroll
            for (int u = 0; u < CH; ++u) a2 = amax2_of(v[u], a2);
            if (three) {
#pragma unroll
                for (int u = 0; u < CH; ++u) mn2 = min_nonzero_m1(v[u], mn2);
            }
            if (prove) {
                // (tiles of a few chunks per lane: the wave's amax, the lane's alone would be a weak bound; all lanes are here)
                uint32_t bound2 = a2;
                if constexpr (kSmall) { const uint32_t a = wave_allmax_u32(fold_max16(a2)); bound2 = a | (a << 16); }
                flushed += certain_flushes<CH>(v, bound2);     // widened tile by tile: 16 bits would hold 2047 tiles of a workgroup
            }
        } else {
            for (int u = 0; u < CH; ++u)
                if (c0 + u * 256 < t.n_chunks) {
                    const u32x4 v = load16(t.x + tensor_chunk_off<STRIDED>(t, c0 + u * 256, t.rm.ld));
                    a2 = amax2_of(v, a2);
                    if (three) mn2 = min_nonzero_m1(v, mn2);
                }
        }
    }
    const uint32_t a = block_allmax_u32(fold_max16(a2), sh4);
    uint32_t mn = 0u;
    if (three) mn = block_allmin_u16(fold_min16(mn2), sh4);
    if (threadIdx.x == 0) t.amax_part[b] = a | (mn << 16);
    if (prove) {
        const uint32_t wf = wave_allsum_u32(flushed);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) sh4[threadIdx.x >> 6] = wf;
        __syncthreads();
        if (threadIdx.x == 0) t.flush_part[b] = (sh4[0] + sh4[1]) + (sh4[2] + sh4[3]);
    }
}
template <bool STRIDED>
__global__ __launch_bounds__(256) void k_tensor_amax_group(GroupTensor g, GroupStats riders, int stats_first, int block0) {
    if ((int)blockIdx.x >= stats_first) { stats_partial_body<256>(riders, (int)blockIdx.x - stats_first); return; }
    tensor_amax_body<STRIDED, kTensorChunksPerThread>(g, (int)blockIdx.x + block0);      // block0: the launch covers a part of the table's operands
}
// What pass A found out about the operand: its amax, and whether the sum of the certain-flush lower bounds proves the BF16
// decision.  Same values in every workgroup that calls it.  All partials are loaded together and one barrier exchanges the wave
// results: every workgroup of pass B waits for this before it can scale anything.
__device__ __forceinline__ uint32_t tensor_pass_a_result(const TensorOp& t, bool& proven) {
    __shared__ uint32_t sha[4];
    __shared__ unsigned long long shf[4];
    const bool prove = t.flush_need != 0ull;
    uint32_t a = 0u;
    unsigned long long f = 0ull;
    for (int i0 = threadIdx.x; i0 < t.n_amax; i0 += 4 * 256) {
        uint32_t av[4], fv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool ok = i0 + u * 256 < t.n_amax;
            const int ic = ok ? i0 + u * 256 : i0;           // always a valid slot: the loads need no branch
            av[u] = t.amax_part[ic];
            fv[u] = prove ? t.flush_part[ic] : 0u;
            fv[u] = ok ? fv[u] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) { a = max(a, av[u] & 0xFFFFu); f += fv[u]; }
    }
    a = wave_allmax_u32(a);
    if (prove) f = wave_allsum_u64(f);
    if ((threadIdx.x & 63) == 0) { sha[threadIdx.x >> 6] = a; shf[threadIdx.x >> 6] = f; }
    __syncthreads();
    proven = prove && (shf[0] + shf[1]) + (shf[2] + shf[3]) >= t.flush_need;
    return max(max(sha[0], sha[1]), max(sha[2], sha[3]));
}
// Where pass A shares the launch (see mor_stream.h): a lane's share of one of its tiles.  An element counts as certain to flush against
// the amax of the tile that its wave holds.
template <bool STRIDED>
__device__ __forceinline__ void tensor_stream_count(const TensorOp& t, int tile, int tid, uint32_t& amax, uint32_t& flushes) {
    constexpr int CH = kTensorChunksPerThread, kTile = 256 * CH;
    const int64_t c_first = (int64_t)tile * kTile;
    const uint32_t valid = (uint32_t)(t.n_chunks - c_first < kTile ? t.n_chunks - c_first : kTile);
    RowPos pos{0u, 0u};
    int64_t row0 = 0;
    if constexpr (STRIDED) row0 = row_tile_first(t.rm, c_first, (uint32_t)tid, pos);
    const BufRsrc rx = STRIDED ? make_buf(t.x + row0 * t.rm.ld) : make_buf_window(t.x + c_first * 8, valid * 16u);
    u32x4 v[CH];
    auto load = [&](auto keep) {
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            uint32_t off = (uint32_t)tid * 16u + u * 4096u;
            if constexpr (STRIDED) { off = row_off<16>(pos, (uint32_t)t.rm.ld * 2u, (uint32_t)tid + u * 256u < valid); row_step(t.rm, pos); }
            v[u] = buf_load16_first<decltype(keep)::value>(rx, off, 0u);
        }
    };
    if (tile >= t.keep_from) load(std::true_type{});
    else load(std::false_type{});
    uint32_t a2 = 0u;
#pragma unroll
    for (int u = 0; u < CH; ++u) a2 = amax2_of(v[u], a2);
    const uint32_t a = wave_allmax_u32(fold_max16(a2));
    amax = max(amax, a);
    if (t.flush_need != 0ull) flushes += certain_flushes<CH>(v, a | (a << 16));
}
struct TensorTold {
    uint32_t* words;
    int polls;
};
// STRIDED: operands with padded leading dimensions (see RowMap).  STREAM: pass A shares the launch, a tile per workgroup.
template <int CRIT, bool FAKE, bool STRIDED, bool STREAM>
__device__ __forceinline__ void tensor_quant_body(const TensorOp& t, int b, const TensorTold& told_by) {
    constexpr int CH = kTensorChunksPerThread, kTile = 256 * CH;
    uint32_t told = 0u;
    const uint32_t* copy = STREAM ? stream_copy(told_by.words, b) : nullptr;
    if constexpr (STREAM) told = agent_load(copy);      // (before the tile's loads, so that it is there before them)
    const uint16_t* __restrict__ x = t.x;
    uint8_t* __restrict__ fp8 = t.o.fp8;
    const int64_t n_chunks = t.n_chunks, n_tiles = t.n_tiles, n_slots = t.n_slots;
    u32x4 bufA[CH];
    const bool wide = STRIDED && t.rm.cpr == 0u;             // chunk by chunk, in the careful path below; pass A proves nothing then
    auto load_tile = [&](u32x4* raw, int64_t tile) {
        const int64_t c0 = tile * kTile + threadIdx.x;
        if constexpr (STREAM && !STRIDED) {
            const int64_t left = n_chunks - tile * kTile;
            const BufRsrc rx = make_buf_window(x + tile * (kTile * 8), (uint32_t)(left < kTile ? left : kTile) * 16u);
#pragma unroll
            for (int u = 0; u < CH; ++u) raw[u] = buf_load16(rx, threadIdx.x * 16u + u * 4096u, 0u);
            return;
        }
        if constexpr (STRIDED) {
            // (wide: a null window, so all chunks read as zeros here; the careful path reads them itself)
            RowPos pos{0u, 0u};
            const int64_t row0 = wide ? 0 : row_tile_first(t.rm, tile * kTile, threadIdx.x, pos);
            const BufRsrc rx = make_buf_window(x + row0 * t.rm.ld, wide ? 0u : 0x7FFFFFFFu);
            const uint32_t row_bytes = (uint32_t)t.rm.ld * 2u;
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                raw[u] = buf_load16(rx, row_off<16>(pos, row_bytes, c0 + u * 256 < n_chunks), 0u);
                row_step(t.rm, pos);
            }
            return;
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int64_t c = c0 + u * 256;
            if (c < n_chunks) raw[u] = load16(x + c * 8);
            else { raw[u].x = 0u; raw[u].y = 0u; raw[u].z = 0u; raw[u].w = 0u; }
        }
    };
    int64_t tl = b;
    load_tile(bufA, tl);
    bool proven;                                             // then the BF16 fallback is written in this sweep
    uint32_t abits;
    if constexpr (STREAM) {
        told = stream_told(copy, told, told_by.polls);
        if (__builtin_expect(told == 0u, 0)) {
            told = stream_scan(told_by.words, (int)n_tiles, stream_scan_from((uint32_t)b, (int)n_tiles), (uint32_t)t.flush_need, [&](int k, int tid, uint32_t& amax, uint32_t& flushes) { tensor_stream_count<STRIDED>(t, k, tid, amax, flushes); });
            asm volatile("" : "+s"(tl));                     // the tile is loaded again, so that its registers need not be kept meanwhile
            load_tile(bufA, tl);
        }
        abits = told & kAmaxBits;
        proven = (told & kToldProven) != 0u;
    } else abits = tensor_pass_a_result(t, proven);
    uint16_t* __restrict__ bf16 = t.o.bf16;
    if (b == 0 && threadIdx.x == 0) { t.abits[0] = abits; t.abits[1] = proven ? 1u : 0u; }
    // one block = the group: under GAM the block's own mantissa is the group mantissa and the scale is s_b
    const uint32_t mode = t.mode;
    const float s = block_scale(abits, kE4M3Max, mode, group_mantissa_bits(abits, kE4M3Max, mode));
    const float s5 = (CRIT == kCritEq3) ? block_scale(abits, kE5M2Max, mode, group_mantissa_bits(abits, kE5M2Max, mode)) : 0.0f;
    const bool fast = abits < fast_amax_limit(mode) && !wide;
    const bool dual = CRIT == kCritEq3 && s5 == 128.0f * s;
    const bool emit = !(proven && (t.flags & kTensorLean) != 0u);             // lean payload: the codes of a proven BF16 operand are not stored
    const float s_inv = FAKE ? 1.0f / s : 0.0f;
    uint16_t* __restrict__ fakep = t.o.fake;     // fake quantization: == bf16, so a proven fallback is already in place
    TensorAcc acc{{0.0f, 0.0f, 0.0f, 0.0f}, 0u};
    // Stores go through bounds-checked buffer windows over the tile (a tail tile's window is shorter; a payload that
    // is not wanted gets a null window), so the quantization sweep has no branches and stays one basic block: with
    // per-lane or per-operand branches around the stores the compiler defers the error terms of all eight chunks
    // and keeps their scaled values in registers.
    auto process = [&](const u32x4* raw, int64_t tile) {
        // Binary32 sums in three short chains instead of one long one: a tile's terms, the tiles of a workgroup, the workgroups
        // (binary64).  Error against 64 bits of an 8192 x 14336 operand, rms over 24 operands: 1.2e-7 with one chain over all
        // tiles, 3.5e-8 with a chain per tile, at the same time per call.  Padded rows start a chain per chunk as well, 2.4e-8 (the
        // rounding of the result is 2.3e-8; 0.5 % of the time): their former kernel, one chunk per lane and tile, had that.
        TileSums sum{0.0f, 0.0f, 0.0f, 0.0f};
        const int64_t c_first = tile * kTile;
        const int64_t c0 = c_first + threadIdx.x;
        const int64_t left = n_chunks - c_first;
        const uint32_t valid = (uint32_t)(left < kTile ? left : kTile);      // chunks of this tile
        int64_t row0 = 0;
        RowPos pos0{0u, 0u};
        if constexpr (STRIDED) row0 = wide ? 0 : row_tile_first(t.rm, c_first, threadIdx.x, pos0);
        const int64_t at8 = STRIDED ? row0 * t.o.ld_fp8 : c_first * 8, atb = STRIDED ? row0 * t.o.ld_bf16 : c_first * 8,
                      atf = STRIDED ? row0 * t.o.ld_fake : c_first * 8;
        const BufRsrc r8 = make_buf_window(fp8 + at8, (FAKE || !emit) ? 0u : (STRIDED ? 0x7FFFFFFFu : valid * 8u));
        const BufRsrc rb = make_buf_window(bf16 + atb, proven ? (STRIDED ? 0x7FFFFFFFu : valid * 16u) : 0u);
        const BufRsrc rf = make_buf_window(fakep + atf, (FAKE && !proven) ? (STRIDED ? 0x7FFFFFFFu : valid * 16u) : 0u);
        const uint32_t off8 = threadIdx.x * 8u, off16 = threadIdx.x * 16u;
        // byte offsets of chunk u in the payload and in the BF16 output; STRIDED lanes beyond the last chunk get none
        RowPos pos = pos0;
        auto at_fp8 = [&](int u) -> uint32_t {
            if constexpr (!STRIDED) return off8 + u * 2048u;
            const uint32_t v = row_off<8>(pos, (uint32_t)t.o.ld_fp8, threadIdx.x + u * 256u < valid);
            row_step(t.rm, pos);
            return v;
        };
        auto at_16 = [&](int u, int64_t ld) -> uint32_t {
            if constexpr (!STRIDED) return off16 + u * 4096u;
            const uint32_t v = row_off<16>(pos, (uint32_t)ld * 2u, threadIdx.x + u * 256u < valid);
            row_step(t.rm, pos);
            return v;
        };
#pragma unroll
        for (int u = 0; u < CH; ++u) acc.zero2 = zero2_of(raw[u], acc.zero2);
        asm volatile("" : "+v"(acc.zero2));      // counted here, not sunk below the sweep (which would keep the masked words alive)
#pragma unroll
        for (int u = 0; u < CH; ++u) buf_store16<kBufStoreNt>(rb, at_16(u, t.o.ld_bf16), raw[u]);       // proven fallback
        pos = pos0;
        if constexpr (STRIDED) asm volatile("" : "+v"(pos.r), "+v"(pos.c));      // the sweep's offsets are formed chunk by chunk, not kept from here
        if (CRIT == kCritEq3 && fast && dual) {
            // both formats in one sweep with one reciprocal per element (see quant8_dual)
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                u32x4 deq;
                TileSums c = STRIDED ? TileSums{0.0f, 0.0f, 0.0f, 0.0f} : sum;
                const u32x2 codes = quant8_dual<FAKE>(raw[u], s, s_inv, c.e0, c.e1, c.f0, c.f1, deq);
                sum = STRIDED ? sum + c : c;
                if constexpr (FAKE) buf_store16<kBufStoreNt>(rf, at_16(u, t.o.ld_fake), deq);
                else buf_store8<kBufStoreNt>(r8, at_fp8(u), 0u, codes);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else if (fast) {
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                u32x4 deq;
                TileSums c = STRIDED ? TileSums{0.0f, 0.0f, 0.0f, 0.0f} : sum;
                const u32x2 codes = quant8_fast_deq<false, FAKE>(raw[u], s, s_inv, c.e0, c.e1, deq);
                if constexpr (FAKE) buf_store16<kBufStoreNt>(rf, at_16(u, t.o.ld_fake), deq);
                else buf_store8<kBufStoreNt>(r8, at_fp8(u), 0u, codes);
                if constexpr (CRIT == kCritEq3) (void)quant8_fast<true>(raw[u], s5, c.f0, c.f1);
                sum = STRIDED ? sum + c : c;
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma clang loop unroll(disable)
            for (int u = 0; u < CH; ++u) {
                const int64_t c = c0 + u * 256;
                if (c < n_chunks) {
                    const uint16_t* __restrict__ src = x + tensor_chunk_off<STRIDED>(t, c, t.rm.ld);
                    sum.e0 += quant8_careful_mem<false>(src, s, (FAKE || !emit) ? nullptr : fp8 + tensor_chunk_off<STRIDED>(t, c, t.o.ld_fp8),
                                                        (FAKE && !proven) ? fakep + tensor_chunk_off<STRIDED>(t, c, t.o.ld_fake) : nullptr, s_inv);
                    if constexpr (CRIT == kCritEq3) sum.f0 += quant8_careful_mem<true>(src, s5, nullptr);
                    if (wide) acc.zero2 = pk_sub_u16(zero2_of(load16(src), acc.zero2), 0x00040004u);       // counted as eight zeros above
                }
            }
        }
        acc.s = acc.s + sum;
    };
    for (;;) {
        process(bufA, tl);
        if constexpr (STREAM) break;
        tl += n_slots;
        if (tl >= n_tiles) break;
        load_tile(bufA, tl);
    }
    TensorPartials tp{t.err, t.err5, t.zero};
    tensor_publish<CRIT>(acc, tp, b);
}
template <int CRIT, bool FAKE, bool STRIDED>
__global__ __launch_bounds__(256) void k_tensor_quant_group(GroupTensor g, int block0) {
    const int block = (int)blockIdx.x + block0;
    const int op = group_find32(g.slot_end, g.n, block);
    tensor_quant_body<CRIT, FAKE, STRIDED, false>(g.op[op], block - (op ? g.slot_end[op - 1] : 0), TensorTold{});
}
// Passes A and B of per-tensor operands under Eq. 2 in one launch (see mor_stream.h).  The first `rider_wgs` workgroups compute the partial
// statistics records of the batch's sub-tensor operands.  The operand's words lie in the array of the E5M2 sums, which Eq. 2 leaves free.
// g.amax_end: groups of the first pass; g.slot_end: workgroups of the second, a tile each, padded to groups of eight.
__device__ __forceinline__ uint32_t* stream_words(const TensorOp& t) { return reinterpret_cast<uint32_t*>(t.err5); }
// Operands that are read once and have no part in the passes -- 128 x 128 blocks, a 1 x 128 operand, the other operands of a layer or of a slice
// -- go through in workgroups spread evenly over the launch: the first pass, which only reads, and the others then overlap.  Their
// table does not fit the kernel arguments with the others; the launch that clears the words puts it into the workspace.
struct TensorFill {
    GroupTeam team;
    GroupSubT<1> sub;
    StatsRec* sub_rec;       // the 1 x 128 operand's records, one per workgroup (nullptr: no statistics)
    float near_tol;
    int32_t sub_blocks;      // its workgroups
};
struct FillOrder {
    Spread sub, team;        // groups of eight workgroups: of the 1 x 128 operand, among the next `early` ones; of the blocks, among the rest
    uint32_t alone;          // groups of the launch before all these
    uint32_t early;
};
enum { kFillNone = 0, kFillFlat = 1, kFillRows = 2 };      // form of the 1 x 128 operand
constexpr int kFillWords = 1024;
static_assert(sizeof(TensorFill) <= 4 * kFillWords, "behind the words of an operand's tiles");
constexpr int kTensorStreamMaxTiles = kStreamMaxTiles - kFillWords;
__device__ __forceinline__ uint32_t* fill_table(uint32_t* words) { return words + kStreamWords - kFillWords; }
struct StreamClear {
    int32_t n, tiles[kMaxGroup];
    uint32_t* words[kMaxGroup];
};
__global__ __launch_bounds__(256) void k_tensor_stream_clear(StreamClear c, TensorFill fill) {      // blockIdx.y = operand, then the table
    if ((int)blockIdx.y < c.n) { stream_clear(c.words[blockIdx.y], c.tiles[blockIdx.y], (int)blockIdx.x); return; }
    const uint32_t* from = reinterpret_cast<const uint32_t*>(&fill);
    if (blockIdx.x == 0)
        for (int i = (int)threadIdx.x; i < (int)(sizeof(TensorFill) / 4); i += 256) fill_table(c.words[0])[i] = from[i];
}
template <int FILL>
__device__ __forceinline__ void fill_body(const TensorFill* __restrict__ fill, bool is_sub, int group, int in8) {
    __shared__ TeamShared sh;
    __shared__ SubStatsShared ssh;
    if (is_sub) {
        const int block = group * 8 + in8, blocks = fill->sub_blocks;
        if (block >= blocks) return;
        StatsRec* rec = fill->sub_rec;
        if (rec) sub_solo_body<kCritEq2, false, FILL == kFillRows>(fill->sub, rec, fill->near_tol, block, blocks, ssh);
        else sub_group_body<kCritEq2, false, false, FILL == kFillRows>(fill->sub, (int64_t)block, (int64_t)blocks, nullptr, 0.0f);
        return;
    }
    const int64_t wg = (int64_t)group * 8 + in8;
    const int n = fill->team.n;
    if (wg >= fill->team.unit_end[n - 1]) return;
    const int op = group_find(fill->team.unit_end, n, wg);
    const TeamOp t = fill->team.op[op];
    team_block<kTeamWg128, kCritEq2, false, false, kTeamAlone>(t, wg - (op ? fill->team.unit_end[op - 1] : 0), sh, StreamUnit{}, [] { return 0u; });
}
template <bool FAKE, bool STRIDED, int FILL>
__global__ __launch_bounds__(256) void k_tensor_stream(GroupTensor g, GroupStats riders, StreamOrder order, int rider_wgs, int polls, FillOrder fo) {
    const int block = (int)blockIdx.x - (rider_wgs + 7) / 8 * 8;
    if (block < 0) {
        if ((int)blockIdx.x < rider_wgs) stats_partial_body<256>(riders, (int)blockIdx.x);
        return;
    }
    uint32_t group = (uint32_t)block >> 3;
    const int in8 = block & 7;
    if constexpr (FILL != kFillNone) {
        if (group >= fo.alone) {
            group -= fo.alone;
            const bool early = group < fo.early;
            const Spread& s = early ? fo.sub : fo.team;
            const uint32_t in_part = early ? group : group - fo.early, before = spread_before(s, in_part);
            if (spread_before(s, in_part + 1u) != before) {
                fill_body<FILL>(reinterpret_cast<const TensorFill*>(fill_table(stream_words(g.op[0]))), early, (int)before, in8);
                return;
            }
            group = fo.alone + group - (early ? before : fo.sub.n + before);
        }
    }
    const StreamPlace place = stream_place(order, group);
    if (place.first) {
        __shared__ uint32_t sh8[8];
        const int op = group_find32(g.amax_end, g.n, (int)place.group);
        const TensorOp& t = g.op[op];
        const int in_op = (int)place.group - (op ? g.amax_end[op - 1] : 0), tiles = (int)t.n_tiles, tile = in_op * 8 + in8;
        auto count = [&](int k, int tid, uint32_t& amax, uint32_t& flushes) { tensor_stream_count<STRIDED>(t, k, tid, amax, flushes); };
        if (tile < tiles) stream_first(stream_words(t), tile, sh8, count);
        else if (in8 == 0 && in_op * 8 >= tiles) (void)stream_collect(stream_words(t), tiles, (uint32_t)t.flush_need, polls, sh8, count);
        return;
    }
    const int wg = (int)place.group * 8 + in8;
    const int op = group_find32(g.slot_end, g.n, wg);
    const TensorOp& t = g.op[op];
    const int b = wg - (op ? g.slot_end[op - 1] : 0);
    if (b >= (int)t.n_tiles) return;
    tensor_quant_body<kCritEq2, FAKE, STRIDED, true>(t, b, TensorTold{stream_words(t), polls});
}
// Decision on a per-tensor operand from its sums (se and se5 over n non-zero elements): every thread of the workgroup calls it and gets
// the mask; with `emit`, thread 0 writes the outputs and the statistics.
template <int CRIT, int T>
__device__ __forceinline__ uint32_t tensor_decide(const TensorOp& t, float near_tol, double se, double se5, unsigned long long n, uint32_t abits,
                                                  bool proven, bool emit) {
    if (abits >= kInfBits) { se = (double)__builtin_inff(); se5 = se; }
    uint32_t mask;
    if constexpr (CRIT == kCritEq3) mask = (se < se5) ? 0u : 1u;
    else mask = ((n ? se / (double)n : 0.0) < (double)t.th) ? 0u : 1u;
    uint32_t amin_bits = 0u;
    if (t.three && mask == 1u) {           // Eq. (4): the operand is kept in E5M2 if its dynamic range fits
        amin_bits = global_amin_bits<T>(t.amax_part, t.n_amax);
        if (range_fits_e5m2(abits, amin_bits, n ? 1u : 0u)) mask = 2u;
    }
    if (emit && threadIdx.x == 0) {
        const KOut& o = t.o;
        const float err_f = (float)se;
        const uint32_t nnz32 = n > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)n;
        const uint32_t mg = group_mantissa_bits(abits, kE4M3Max, t.mode), mg5 = group_mantissa_bits(abits, kE5M2Max, t.mode);
        const float s = mask == 2u ? block_scale(abits, kE5M2Max, t.mode, mg5) : block_scale(abits, kE4M3Max, t.mode, mg);
        if (t.three && o.amin) o.amin[0] = __uint_as_float(amin_bits << 16);
        o.scale[0] = s;
        if (t.mode != kScaleFp32 && o.e8m0) o.e8m0[0] = (uint8_t)(__float_as_uint(s) >> 23);
        if (t.mode != kScaleFp32 && o.gmant) { o.gmant[0] = mg; o.gmant[1] = mg5; }
        o.amax[0] = __uint_as_float(abits << 16);
        o.err_sum[0] = err_f;
        o.nnz[0] = nnz32;
        if constexpr (CRIT == kCritEq3) o.err5_sum[0] = (float)se5;
        o.mask[0] = (uint8_t)mask;
        if (t.stats) {     // statistics of a one-block operand, same arithmetic as k_stats_single
            StatsDev* st = t.stats;
            const float metric = nnz32 ? err_f / (float)nnz32 : 0.0f;
#pragma unroll
            for (int k = 0; k < 12; ++k) st->hist[k] = 0u;
            st->hist[stats_bin(metric)] = 1u;
            const bool near = fabs((double)metric - (double)t.th) <= (double)near_tol * (double)t.th;
            const unsigned long long total = (unsigned long long)t.n_chunks * 8ull;
            stats_finish(st, 1, total, (double)err_f, nnz32, mask == 1u ? 1ull : 0ull, near ? 1ull : 0ull, mask == 2u ? 1ull : 0ull,
                         mask == 1u ? total : 0ull, mask == 2u ? total : 0ull, proven && (t.flags & kTensorReport) != 0u ? 1u : 0u);
        }
    }
    return mask;
}
template <int CRIT, bool STRIDED>
__device__ __forceinline__ void tensor_finish_body(const GroupTensor& g, int block) {
    const int op = group_find32(g.copy_end, g.n, block);
    const TensorOp& t = g.op[op];
    const int b = block - (op ? g.copy_end[op - 1] : 0);
    const int nb = g.copy_end[op] - (op ? g.copy_end[op - 1] : 0);
    const bool proven = t.abits[1] != 0u;                     // pass B already wrote the fallback
    if (proven && b != 0) return;                             // only the operand's first workgroup has work left
    __shared__ double shd[4];
    __shared__ unsigned long long shl[4];
    double se = 0.0, se5 = 0.0;
    unsigned long long sz = 0;
    tensor_partial_sums<CRIT>(t.err, t.err5, t.zero, t.n_slots, se, se5, sz);
    se = block_sum_shfl<double>(se, shd);
    sz = block_sum_shfl<unsigned long long>(sz, shl);
    if constexpr (CRIT == kCritEq3) se5 = block_sum_shfl<double>(se5, shd);
    const uint32_t abits = t.abits[0];
    const unsigned long long n_padded = (unsigned long long)t.n_tiles * kTensorChunksPerBlock * 8;
    const uint32_t mask = tensor_decide<CRIT, 256>(t, g.near_tol, se, se5, n_padded - sz, abits, proven, b == 0);
    if (mask == 2u) {
        const bool fast = abits < fast_amax_limit(t.mode);
        const float s5 = block_scale(abits, kE5M2Max, t.mode, group_mantissa_bits(abits, kE5M2Max, t.mode));
        uint16_t* __restrict__ fakep = t.o.fake;
        const float s_inv = fakep ? 1.0f / s5 : 0.0f;
        for (int64_t c = (int64_t)b * 256 + threadIdx.x; c < t.n_chunks; c += (int64_t)nb * 256)
            requant_chunk_e5m2(t.x + tensor_chunk_off<STRIDED>(t, c, t.rm.ld), fakep ? nullptr : t.o.fp8 + tensor_chunk_off<STRIDED>(t, c, t.o.ld_fp8),
                               fakep ? fakep + tensor_chunk_off<STRIDED>(t, c, t.o.ld_fake) : nullptr, s5, s_inv, fast);
        return;
    }
    if (proven || mask == 0u || t.o.bf16 == nullptr) return;
    if constexpr (STRIDED) {
        const int64_t stride = (int64_t)nb * 256;
        int64_t c = (int64_t)b * 256 + threadIdx.x;
        for (; c + 3 * stride < t.n_chunks; c += 4 * stride) {
            u32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = load16(t.x + tensor_chunk_off<STRIDED>(t, c + u * stride, t.rm.ld));
#pragma unroll
            for (int u = 0; u < 4; ++u) store16(t.o.bf16 + tensor_chunk_off<STRIDED>(t, c + u * stride, t.o.ld_bf16), v[u]);
        }
        for (; c < t.n_chunks; c += stride)
            store16(t.o.bf16 + tensor_chunk_off<STRIDED>(t, c, t.o.ld_bf16), load16(t.x + tensor_chunk_off<STRIDED>(t, c, t.rm.ld)));
    } else {
        copy_chunk_tiles(t.x, t.o.bf16, t.n_chunks, b, nb);
    }
}
// ---- a small operand alone in its call: two launches instead of three.  The workgroups of pass B keep their tile in registers, leave
//      their sums and draw a ticket; the last one decides for the operand and tells the others, which copy their tile if it stays in
//      BF16 after all (or rewrite it in E5M2).  Nobody waits without end: a workgroup that is not told in time (others may not have
//      found a place on the chip) says so, looks once more and leaves; the one that decides tells first and then looks who has left,
//      so that at least one of the two sees to the tile (if both do, they store the same bytes).  Beside another stream's matrix
//      products that fill the chip (8192 x 8192 x 8192 in BF16), where every launch waits for places, 9 calls of 1024 x 1024 end in the
//      10.4 ms of twelve products, 3 with three launches, and the longest takes 1.5 ms (2.7); the products take 0 to 3 % longer.
//      Beside copies of 1 GiB, and beside three streams of such calls, all calls take less than with three launches.
constexpr int kTicketGroup = 16;             // workgroups to a first ticket; tickets of one address complete some 15 ns apart
constexpr int kOneMaxSlots = 512;
constexpr int kOneLine = 32;                 // words: a line of its own for every ticket and every copy of the decision
constexpr int kTicketRoot = kOneMaxSlots / kTicketGroup * kOneLine;
constexpr int kOneToldCopies = 32;           // of the decision, so that few workgroups look at one line
constexpr int kOneTold = kTicketRoot + kOneLine, kOneLeft = kOneTold + kOneToldCopies * kOneLine, kOneSyncWords = kOneLeft + kOneMaxSlots;
enum : uint32_t { kToldNothing = 0u, kToldMask = 1u };      // kToldMask + the mask
static_assert(8192 + kOneSyncWords <= kMaxQuantBlocks && kOneMaxSlots <= 8192, "the words lie behind the zero counts in their array");
__device__ __forceinline__ uint32_t* one_sync(const TensorOp& t) { return t.zero + 8192; }
template <int T>             // lanes of the workgroup (as a constant: blockDim is read from memory, 0.25 us)
__device__ __forceinline__ void clear_one_sync(const TensorOp& t) {
    uint32_t* sync = one_sync(t);
    for (uint32_t i = blockIdx.x * (uint32_t)T + threadIdx.x; i < (uint32_t)kOneSyncWords; i += gridDim.x * (uint32_t)T) sync[i] = 0u;
}
__global__ __launch_bounds__(256) void k_tensor_amax_one(OneTensor g) {      // padded rows
    clear_one_sync<256>(g.op[0]);
    tensor_amax_body<true, kSmallChunksPerThread>(g, (int)blockIdx.x);
}
// Dense rows: a workgroup takes a tile of the grouped kernels and counts certain flushes as they do, so that the proof (which the statistics
// report, and which leaves out a lean operand's payload) does not depend on the kernel: a chunk's bound is the amax of the eight chunks that
// one lane of theirs takes, here spread over Q lanes that exchange it, and counted are lanes whose eight chunks all exist.
template <int T, int CH>
__global__ __launch_bounds__(T) void k_tensor_amax_one_dense(OneTensor g) {
    constexpr int Q = T / 256, NW = T / 64;
    static_assert(T * CH == kTensorChunksPerBlock, "a tile of the grouped kernels");
    __shared__ uint32_t lane_max[Q][256], sha[NW], shm[NW], shf[NW];
    const TensorOp& t = g.op[0];
    clear_one_sync<T>(t);
    const int tid = threadIdx.x, w = tid >> 6, q = tid >> 8, l = tid & 255;
    const int64_t c_first = (int64_t)blockIdx.x * kTensorChunksPerBlock;
    const uint32_t valid = (uint32_t)(t.n_chunks - c_first < kTensorChunksPerBlock ? t.n_chunks - c_first : kTensorChunksPerBlock);
    const BufRsrc rx = make_buf(t.x + c_first * 8);
    const uint32_t first = (uint32_t)(q * CH * 256 + l);                            // this lane's first chunk in the tile, then 256 further
    u32x4 v[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) v[u] = buf_load16_first<true>(rx, off_if(first + u * 256u < valid, (first + u * 256u) * 16u), 0u);
    uint32_t a2 = 0u, mn2 = 0xFFFFFFFFu, flushed = 0u;
#pragma unroll
    for (int u = 0; u < CH; ++u) a2 = amax2_of(v[u], a2);
    if (t.three) {
#pragma unroll
        for (int u = 0; u < CH; ++u) mn2 = min_nonzero_m1(v[u], mn2);
    }
    if (t.flush_need != 0ull) {
        lane_max[q][l] = a2;
        __syncthreads();
        uint32_t bound2 = 0u;
#pragma unroll
        for (int k = 0; k < Q; ++k) bound2 = pk_max_u16(bound2, lane_max[k][l]);
        flushed = (uint32_t)l + (kTensorChunksPerThread - 1) * 256u < valid ? certain_flushes<CH>(v, bound2) : 0u;
    }
    const uint32_t a_w = wave_allmax_u32(fold_max16(a2)), m_w = wave_allmax_u32(0xFFFFu - fold_min16(mn2)), f_w = wave_allsum_u32(flushed);
    if ((tid & 63) == 0) { sha[w] = a_w; shm[w] = m_w; shf[w] = f_w; }
    __syncthreads();
    if (tid != 0) return;
    uint32_t a = 0u, m = 0u, f = 0u;
#pragma unroll
    for (int k = 0; k < NW; ++k) { a = max(a, sha[k]); m = max(m, shm[k]); f += shf[k]; }
    t.amax_part[blockIdx.x] = a | (t.three ? (0xFFFFu - m) << 16 : 0u);
    t.flush_part[blockIdx.x] = f;
}
// T lanes with CH chunks each.  Dense operands: a tile is the 2048 chunks that 256 lanes take in the grouped kernels, and the sums are
// those of the grouped kernels bit for bit: two lanes that hold a chain of additions in halves hand it on through shared memory.
template <int CRIT, bool FAKE, int T, int CH>
__global__ __launch_bounds__(T, 4) void k_tensor_quant_one(OneTensor g, int polls) {
    constexpr int Q = T / 256, NW = T / 64, kTile = T * CH;
    __shared__ float4 run[256];
    __shared__ float shf[8];
    __shared__ uint32_t sha[NW], shz[NW], sh_last, sh_told, sh_left[kOneMaxSlots / 32];
    __shared__ unsigned long long shl[NW];
    __shared__ double shd[8];
    const TensorOp& t = g.op[0];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, q = tid >> 8, l = tid & 255;
    const int b = (int)blockIdx.x, n_slots = (int)gridDim.x;                        // a tile each
    const int64_t c_first = (int64_t)b * kTile, n_chunks = t.n_chunks;
    const uint32_t first = (uint32_t)(q * CH * 256 + l);                            // this lane's first chunk in the tile, then 256 further
    const uint32_t valid = (uint32_t)(n_chunks - c_first < kTile ? n_chunks - c_first : kTile);
    const bool wide = t.rm.cpr == 0u;
    uint32_t* sync = one_sync(t);
    uint32_t* told_at = sync + kOneTold + (b % kOneToldCopies) * kOneLine;
    auto chunk_off = [&](int64_t c, int64_t ld) -> int64_t {
        if (wide) return tensor_chunk_off<true>(t, c, ld);
        const uint32_t r = row_div(t.rm, (uint32_t)c);        // (an operand that comes here has fewer than 2^31 chunks)
        return (int64_t)r * ld + (int64_t)((uint32_t)c - r * t.rm.cpr) * 8;
    };
    // ---- the tile
    u32x4 raw[CH];
    RowPos pos0{0u, 0u};
    const int64_t row0 = wide ? 0 : row_tile_first(t.rm, c_first, first, pos0);
    if (!wide) {
        const BufRsrc rx = make_buf(t.x + row0 * t.rm.ld);
        RowPos pos = pos0;
#pragma unroll
        for (int u = 0; u < CH; ++u) { raw[u] = buf_load16(rx, row_off<16>(pos, (uint32_t)t.rm.ld * 2u, first + u * 256u < valid), 0u); row_step(t.rm, pos); }
    } else {
#pragma unroll
        for (int u = 0; u < CH; ++u)
            raw[u] = first + u * 256u < valid ? load16(t.x + chunk_off(c_first + first + u * 256u, t.rm.ld)) : u32x4{0u, 0u, 0u, 0u};
    }
    // ---- what pass A found out
    uint32_t abits = 0u;
    unsigned long long fl = 0ull;
#pragma unroll
    for (int k = 0; k < kAmaxOneTile / T + (kAmaxOneTile % T ? 1 : 0); ++k) {
        const int i = tid + k * T, ic = i < t.n_amax ? i : t.n_amax - 1;              // always a valid slot: the loads need no branch
        const uint32_t av = t.amax_part[ic], fv = t.flush_need ? t.flush_part[ic] : 0u;
        abits = max(abits, av & 0xFFFFu);
        fl += i < t.n_amax ? fv : 0u;
    }
    abits = wave_allmax_u32(abits);
    fl = wave_allsum_u64(fl);
    if (lane == 0) { sha[w] = abits; shl[w] = fl; }
    __syncthreads();
    fl = 0ull;
#pragma unroll
    for (int k = 0; k < NW; ++k) { abits = max(abits, sha[k]); fl += shl[k]; }
    const bool proven = t.flush_need != 0ull && fl >= t.flush_need;                  // then the BF16 fallback is written here
    if (b == 0 && tid == 0) { t.abits[0] = abits; t.abits[1] = proven ? 1u : 0u; }
    const uint32_t mode = t.mode;
    const float s = block_scale(abits, kE4M3Max, mode, group_mantissa_bits(abits, kE4M3Max, mode));
    const float s5 = (CRIT == kCritEq3) ? block_scale(abits, kE5M2Max, mode, group_mantissa_bits(abits, kE5M2Max, mode)) : 0.0f;
    const bool fast = abits < fast_amax_limit(mode) && !wide, dual = CRIT == kCritEq3 && s5 == 128.0f * s;
    const bool emit = !(proven && (t.flags & kTensorLean) != 0u), dense = (t.flags & kTensorDense) != 0u;
    const float s_inv = FAKE ? 1.0f / s : 0.0f;
    const BufRsrc r8 = make_buf_window(t.o.fp8 + row0 * t.o.ld_fp8, (FAKE || !emit || wide) ? 0u : 0x7FFFFFFFu);
    const BufRsrc rb = make_buf_window(t.o.bf16 + row0 * t.o.ld_bf16, proven ? 0x7FFFFFFFu : 0u);
    const BufRsrc rf = make_buf_window(t.o.fake + row0 * t.o.ld_fake, (FAKE && !proven && !wide) ? 0x7FFFFFFFu : 0u);
    // ---- quantize: codes or values stored, terms kept (one lane has its whole chain only if Q is 1)
    uint32_t z2 = 0u;
    float e[CH][8], f[CH][8];
    RowPos pos = pos0;
#pragma unroll
    for (int u = 0; u < CH; ++u) {
        const bool live = first + u * 256u < valid;
        z2 = zero2_of(raw[u], z2);
        u32x4 deq;
        u32x2 codes{0u, 0u};
        if (fast) {
            if (CRIT == kCritEq3 && dual) {
                codes = quant8_dual_terms<FAKE>(raw[u], s, s_inv, e[u], f[u], deq);
            } else {
                codes = quant8_terms<false, FAKE>(raw[u], s, s_inv, e[u], deq);
                if constexpr (CRIT == kCritEq3) { u32x4 none; (void)quant8_terms<true, false>(raw[u], s5, 0.0f, f[u], none); }
            }
            buf_store16<kBufStoreNt>(rb, row_off<16>(pos, (uint32_t)t.o.ld_bf16 * 2u, live), raw[u]);       // proven fallback
            if constexpr (FAKE) buf_store16<kBufStoreNt>(rf, row_off<16>(pos, (uint32_t)t.o.ld_fake * 2u, live), deq);
            else buf_store8<kBufStoreNt>(r8, row_off<8>(pos, (uint32_t)t.o.ld_fp8, live), 0u, codes);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) { e[u][j] = 0.0f; f[u][j] = 0.0f; }
            if (live) {
                const int64_t c = c_first + first + u * 256u;
                const uint16_t* src = t.x + chunk_off(c, t.rm.ld);
                e[u][0] = quant8_careful_mem<false>(src, s, (FAKE || !emit) ? nullptr : t.o.fp8 + chunk_off(c, t.o.ld_fp8),
                                                    (FAKE && !proven) ? t.o.fake + chunk_off(c, t.o.ld_fake) : nullptr, s_inv);
                if constexpr (CRIT == kCritEq3) f[u][0] = quant8_careful_mem<true>(src, s5, nullptr);
                if (proven) store16(t.o.bf16 + chunk_off(c, t.o.ld_bf16), raw[u]);
            }
        }
        row_step(t.rm, pos);
    }
    // ---- sums: dense operands in one chain per lane of 256, padded ones chunk by chunk (as the grouped kernels)
    TileSums sum{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        if (q == k) {
            if (k > 0) { const float4 v = run[l]; sum = TileSums{v.x, v.y, v.z, v.w}; }
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                TileSums c = dense ? sum : TileSums{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    c.e0 += e[u][2 * j]; c.e1 += e[u][2 * j + 1];
                    if constexpr (CRIT == kCritEq3) { c.f0 += f[u][2 * j]; c.f1 += f[u][2 * j + 1]; }
                }
                sum = dense ? c : sum + c;
            }
            if (k + 1 < Q) run[l] = float4{sum.e0, sum.e1, sum.f0, sum.f1};
        }
        if (k + 1 < Q) __syncthreads();
    }
    const uint32_t z_w = wave_allsum_u32(fold_add16(z2));
    if (lane == 0) shz[w] = z_w;
    if (q == Q - 1) {
        const float e_w = wave_allsum_f32(sum.e0 + sum.e1);
        float e5_w = 0.0f;
        if constexpr (CRIT == kCritEq3) e5_w = wave_allsum_f32(sum.f0 + sum.f1);
        if (lane == 0) { shf[w & 3] = e_w; shf[4 + (w & 3)] = e5_w; }
    }
    __syncthreads();
    // ---- ticket
    if (tid == 0) {
        uint32_t z = 0u;
#pragma unroll
        for (int k = 0; k < NW; ++k) z += shz[k];
        agent_store(t.err + b, (shf[0] + shf[1]) + (shf[2] + shf[3]));
        agent_store(t.zero + b, z);
        if constexpr (CRIT == kCritEq3) agent_store(t.err5 + b, (shf[4] + shf[5]) + (shf[6] + shf[7]));
        wait_memory();                                        // the sums have arrived before the ticket is drawn
        const uint32_t grp = (uint32_t)b / kTicketGroup, n_grp = (uint32_t)(n_slots + kTicketGroup - 1) / kTicketGroup;
        const uint32_t in_grp = (uint32_t)n_slots - grp * kTicketGroup < kTicketGroup ? (uint32_t)n_slots - grp * kTicketGroup : kTicketGroup;
        bool last = __hip_atomic_fetch_add(sync + grp * kOneLine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == in_grp - 1u;
        if (last) last = __hip_atomic_fetch_add(sync + kTicketRoot, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n_grp - 1u;
        sh_last = last ? 1u : 0u;
    }
    __syncthreads();
    const bool decides = sh_last != 0u, open = !proven && (t.o.bf16 != nullptr || t.three != 0u);      // open: the decision may ask for one more store
    // What the decision asks for in one tile: the BF16 fallback (from the registers where they hold it), or the E5M2 payload.
    auto finish_tile = [&](uint32_t mask, int tile, bool held) {
        const bool fast5 = abits < fast_amax_limit(mode);
        const float sc5 = block_scale(abits, kE5M2Max, mode, group_mantissa_bits(abits, kE5M2Max, mode)), inv5 = FAKE ? 1.0f / sc5 : 0.0f;
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int64_t c = (int64_t)tile * kTile + first + u * 256;
            if (c >= n_chunks) continue;
            const uint16_t* src = t.x + chunk_off(c, t.rm.ld);
            if (mask == 2u) requant_chunk_e5m2(src, FAKE ? nullptr : t.o.fp8 + chunk_off(c, t.o.ld_fp8), FAKE ? t.o.fake + chunk_off(c, t.o.ld_fake) : nullptr, sc5, inv5, fast5);
            else if (t.o.bf16) store16(t.o.bf16 + chunk_off(c, t.o.ld_bf16), held ? raw[u] : load16(src));
        }
    };
    if (!decides) {
        if (!open) return;
        if (tid == 0) {
            uint32_t told = kToldNothing;
            for (int poll = 0; poll < polls && told == kToldNothing; ++poll) {
                told = agent_load(told_at);
                if (told == kToldNothing) __builtin_amdgcn_s_sleep(8);
            }
            sh_told = told;
        }
        __syncthreads();
        uint32_t told = sh_told;
        if (told == kToldNothing) {                            // (uniform) what this workgroup has stored comes before the word that it left
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __syncthreads();
            if (tid == 0) {
                agent_store(sync + kOneLeft + b, 1u);
                wait_memory();
                sh_told = agent_load(told_at);
            }
            __syncthreads();
            told = sh_told;
            if (told == kToldNothing) return;
        }
        if (told != kToldMask) finish_tile(told - kToldMask, b, true);
        return;
    }
    // (256 lanes, in the order of the finish pass of the grouped kernels)
    double se = 0.0, se5 = 0.0;
    unsigned long long sz = 0;
    if (q == 0) {
#pragma unroll
        for (int k = 0; k < kOneMaxSlots / 256; ++k) {
            const int i = l + k * 256, ic = i < n_slots ? i : n_slots - 1;            // always a valid slot: the loads need no branch
            const float ev = agent_load(t.err + ic), e5v = CRIT == kCritEq3 ? agent_load(t.err5 + ic) : 0.0f;
            const uint32_t zv = agent_load(t.zero + ic);
            se += i < n_slots ? (double)ev : 0.0; se5 += i < n_slots ? (double)e5v : 0.0; sz += i < n_slots ? zv : 0u;
        }
#pragma unroll
        for (int m = 32; m > 0; m >>= 1) {
            se += __shfl_xor(se, m, 64);
            if constexpr (CRIT == kCritEq3) se5 += __shfl_xor(se5, m, 64);
            sz += __shfl_xor(sz, m, 64);
        }
        if (lane == 0) { shd[w] = se; shd[4 + w] = se5; shl[w] = sz; }
    }
    __syncthreads();
    se = (shd[0] + shd[1]) + (shd[2] + shd[3]);
    se5 = (shd[4] + shd[5]) + (shd[6] + shd[7]);
    sz = (shl[0] + shl[1]) + (shl[2] + shl[3]);
    const unsigned long long n_padded = (unsigned long long)n_slots * kTile * 8;
    const uint32_t mask = tensor_decide<CRIT, T>(t, g.near_tol, se, se5, n_padded - sz, abits, proven, true);
    if (!open) return;
    if (tid < kOneToldCopies) agent_store(sync + kOneTold + tid * kOneLine, kToldMask + mask);
    if (mask == 0u) return;
    finish_tile(mask, b, true);
    wait_memory();
    if (tid < kOneMaxSlots / 32) sh_left[tid] = 0u;
    __syncthreads();                                           // (the decision has been told: the wave that stored it has waited)
    for (int i = tid; i < n_slots; i += T)
        if (agent_load(sync + kOneLeft + i) != 0u) atomicOr(&sh_left[i >> 5], 1u << (i & 31));
    __syncthreads();
    unsigned long long some = __ballot(lane < kOneMaxSlots / 32 && sh_left[lane & (kOneMaxSlots / 32 - 1)] != 0u);
    for (; some; some &= some - 1ull) {                        // 32 tiles each (the same in every wave)
        const int i0 = (__ffsll(some) - 1) * 32;
        for (uint32_t left = sh_left[i0 >> 5]; left; left &= left - 1u) finish_tile(mask, i0 + __ffs((int)left) - 1, false);
    }
}
// Workgroups from `stats_first` on combine the riders' partial statistics records (one workgroup per operand).
template <int CRIT, bool STRIDED>
__global__ __launch_bounds__(256) void k_tensor_finish_group(GroupTensor g, GroupStats riders, int stats_first) {
    if ((int)blockIdx.x >= stats_first) { stats_final_body(riders, (int)blockIdx.x - stats_first); return; }
    tensor_finish_body<CRIT, STRIDED>(g, (int)blockIdx.x);
}
// The same where operands went along (see TensorFill).  `direct`: operands of the table, one bit each, whose statistics are still to be taken,
// by one workgroup; then the 1 x 128 operand of `solo`.  A kernel of its own, since the additional branches' registers and LDS hold up the
// other calls' some 2000 workgroups: per-tensor operands of 744 x 280 and 243 x 456 15.5 us per call without them, 16.4 with, three of 1024 x 1024
// 16.1, 18.0, eight of 512 x 512 16.5, 18.5.
template <bool STRIDED>
__global__ __launch_bounds__(256) void k_tensor_finish_fill(GroupTensor g, GroupStats riders, int stats_first, uint32_t direct, SoloStats solo) {
    if ((int)blockIdx.x >= stats_first) {
        const int op = (int)blockIdx.x - stats_first;
        if (op >= riders.n) solo_final_body<256>(solo);
        else if ((direct >> op) & 1u) stats_partial_body<256>(riders, op ? riders.wg_end[op - 1] : 0);
        else stats_final_body(riders, op);
        return;
    }
    tensor_finish_body<kCritEq2, STRIDED>(g, (int)blockIdx.x);
}
// Group loop of Algorithm 1 for sub-tensor operands: the operand's amax (partials of pass A) gives the
// group mantissas for E4M3 and E5M2, which the block kernels read; also written to the caller's output.
// (E8M0-only operands have a zero mantissa, which their block kernels know.)
struct GamOp {
    const uint32_t* amax_part; int n_amax;
    uint32_t mode;
    uint32_t* gam;         // [4] workspace words read by the block kernels: the two mantissas, then 1 if the pre-pass proved
                           // the tensor-level BF16 decision
    uint32_t* gmant;       // caller's group-mantissa output, may be nullptr
    const uint32_t* flush_part;          // [n_amax] certain flushes counted by the pre-pass, or nullptr
    unsigned long long flush_need;       // that many prove the decision
    uint32_t skip;                       // per-channel columns under GAM: the step that forms their scales derives the mantissas
};
struct GroupGam {
    int n;
    GamOp op[kMaxGroup];
};
// One workgroup per operand, on the critical path of the call: 1024 lanes, four partials of each kind in flight per lane (an
// operand of 2048 partials took 8.7 us with 256 lanes and one load at a time).
constexpr int kGamThreads = 1024;
__global__ __launch_bounds__(kGamThreads) void k_gam_prepare(GroupGam g) {
    __shared__ uint32_t sha[kGamThreads / 64];
    __shared__ unsigned long long shl[kGamThreads / 64];
    const GamOp& t = g.op[blockIdx.x];
    if (t.skip) return;                  // uniform over the workgroup
    uint32_t a = 0u;
    unsigned long long fl_wg = 0ull;
    for (int i0 = threadIdx.x; i0 < t.n_amax; i0 += 4 * kGamThreads) {
        uint32_t av[4], fv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * kGamThreads;
            const int ic = i < t.n_amax ? i : i0;          // always a valid slot: the loads need no branch
            av[u] = t.amax_part[ic];
            fv[u] = t.flush_part ? t.flush_part[ic] : 0u;
            if (i >= t.n_amax) fv[u] = 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) { a = max(a, av[u] & 0xFFFFu); fl_wg += fv[u]; }
    }
    a = wave_allmax_u32(a);
    fl_wg = wave_allsum_u64(fl_wg);
    if ((threadIdx.x & 63) == 0) { sha[threadIdx.x >> 6] = a; shl[threadIdx.x >> 6] = fl_wg; }
    __syncthreads();
    if (threadIdx.x != 0) return;
    unsigned long long flushes = 0ull;
#pragma unroll
    for (int w = 0; w < kGamThreads / 64; ++w) { a = max(a, sha[w]); flushes += shl[w]; }
    t.gam[2] = (t.flush_part && flushes >= t.flush_need) ? 1u : 0u;
    const uint32_t mg = group_mantissa_bits(a, kE4M3Max, t.mode);
    t.gam[0] = mg;
    const uint32_t mg5 = group_mantissa_bits(a, kE5M2Max, t.mode);
    t.gam[1] = mg5;
    if (t.gmant) { t.gmant[0] = mg; t.gmant[1] = mg5; }
}

// Group loop of Algorithm 1 with bands of rows as groups: workgroup (band, w) scans its share of the band's 16-byte chunks,
// then one lane per band turns the band's amax into its two mantissas (table behind the four header words of `gam`).
template <bool KEEP>
__global__ __launch_bounds__(256) void k_band_amax(const uint16_t* __restrict__ x, KShape sh, int64_t group_rows, int wpb,
                                                   uint32_t* __restrict__ part) {
    __shared__ uint32_t sh4[4];
    const int64_t band = blockIdx.x / wpb;
    const int w = blockIdx.x - (int)band * wpb;
    const int64_t r_first = band * group_rows;
    const int64_t n_rows = sh.rows - r_first < group_rows ? sh.rows - r_first : group_rows;
    const int64_t cpr = sh.cols / 8, n_chunks = n_rows * cpr;
    uint32_t a2 = 0u;
    for (int64_t c = (int64_t)w * 256 + threadIdx.x; c < n_chunks; c += (int64_t)wpb * 256) {
        const int64_t r = c / cpr, cc = c - r * cpr;
        const uint16_t* p = x + (r_first + r) * sh.ld + cc * 8;
        a2 = amax2_of(KEEP ? *reinterpret_cast<const u32x4*>(p) : load16(p), a2);
    }
    const uint32_t a = block_allmax_u32(fold_max16(a2), sh4);
    if (threadIdx.x == 0) part[blockIdx.x] = a;
}
__global__ __launch_bounds__(256) void k_gam_prepare_bands(const uint32_t* __restrict__ part, int wpb, int64_t n_groups,
                                                           uint32_t* __restrict__ gam, uint32_t* __restrict__ gmant) {
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x < kGamHeaderWords) gam[threadIdx.x] = 0u;     // no single mantissa, nothing proven
    if (g >= n_groups) return;
    uint32_t a = 0u;
    for (int k = 0; k < wpb; ++k) a = max(a, part[g * wpb + k]);
    const uint32_t mg = group_mantissa_bits(a, kE4M3Max, kScaleGam), mg5 = group_mantissa_bits(a, kE5M2Max, kScaleGam);
    gam[kGamHeaderWords + 2 * g] = mg; gam[kGamHeaderWords + 2 * g + 1] = mg5;
    if (gmant) { gmant[2 * g] = mg; gmant[2 * g + 1] = mg5; }
}

// ======================================================================================
// Launchers
// ======================================================================================
static inline size_t align16(size_t v) { return (v + 15) & ~(size_t)15; }
// Workgroups per band of the band-amax pass: about 2048 in all, at most one per 8 KB of the band.
static int band_wgs(const BatchItem& it) {
    const int64_t n_groups = (it.sh.rows + it.group_rows - 1) / it.group_rows;
    int64_t per = 2048 / n_groups, cap = (it.group_rows * it.sh.cols + 4095) / 4096;
    if (per > cap) per = cap;
    return (int)(per < 1 ? 1 : per);
}


TensorPlan plan_tensor(int64_t, int64_t) {
    TensorPlan pl;
    pl.amax_blocks = kAmaxOneTile;
    pl.quant_blocks = kMaxQuantBlocks;
    size_t off = 0;
    pl.off_amax_part = off; off = align16(off + sizeof(uint32_t) * (size_t)pl.amax_blocks);
    pl.off_err_part = off;  off = align16(off + sizeof(float) * (size_t)pl.quant_blocks);
    pl.off_err5_part = off; off = align16(off + sizeof(float) * (size_t)pl.quant_blocks);
    pl.off_nnz_part = off;  off = align16(off + sizeof(uint32_t) * (size_t)pl.quant_blocks);   // zero counts
    pl.off_decision = off;  off = align16(off + 16);                                           // [0] global amax bits
    pl.off_flush_part = off; off = align16(off + sizeof(uint32_t) * (size_t)pl.amax_blocks);   // certain-flush lower bounds
    pl.bytes = off;
    return pl;
}

LeftWords lone_tensor_left_words() { return {plan_tensor(0, 0).off_nnz_part + sizeof(uint32_t) * (8192 + kOneLeft), kOneMaxSlots}; }

size_t scope_workspace_bytes(int64_t) { return align16(3 * sizeof(double) * kScopeBlocks + 16); }

static bool is_flat(const KShape& sh, const KOut& o) {
    return sh.ld == sh.cols && o.ld_fp8 == sh.cols && (o.bf16 == nullptr || o.ld_bf16 == sh.cols) &&
           (o.fake == nullptr || o.ld_fake == sh.cols);
}
constexpr int64_t kSubRiderMaxUnits = 16384;  // 1x128 operands of at most 128 MiB ride on a team launch; larger ones run faster uncapped
constexpr int64_t kSubFlatMaxBlocks = 1536;   // workgroups of 4 waves, each wave strides over 8 KB units: 6 per compute unit is what the kernel's
                                              // registers let be resident, so no workgroup waits for another to end (one 64 MiB operand, cold
                                              // caches: 21.0 us at 1536 against 23.2 us at 2048 (one unit per wave); 112 MiB: 32.1 against 34.5 us;
                                              // 224 MiB: 65 us either way)
constexpr int64_t kSubRowsAlone = 81920;      // us per call, general kernel / ROWS form: 33 000 blocks 6.1 / 7.8 (dense with a tail), 6.1 / 6.8
                                              // (padded), 7.0 / 8.2 (ragged); 66 000 blocks 9.7 / 10.5, 9.5 / 8.8, 11.4 / 11.2; 77 000 blocks 10.9 / 11.2
                                              // (padded); 82 500 blocks 11.6 / 11.1 (tail); 93 000 blocks 12.9 / 11.5, 12.7 / 11.5, 15.6 / 12.1.  Several
                                              // operands share the launch: twelve of 64 to 2048 rows 53 to 78 us per call / 19 to 39
constexpr int64_t kSubRowsMaxBlocks = 1280;   // the ROWS form's registers (90) let five be resident per compute unit
static int clamp_grid_y(int64_t v) { return (int)(v < 1 ? 1 : (v > 65535 ? 65535 : v)); }

// The general 1 x 128 kernel: one operand per launch.
template <int CRIT>
static void launch_sub1x128_crit(const dim3& grid, const uint16_t* x, const KShape& sh, const KOut& o, bool defer, float th,
                                 uint32_t mode, const uint32_t* gam, uint32_t three, uint32_t group_rows, hipStream_t st) {
    const bool fake = o.fake != nullptr;
    if (defer) {
        if (fake) k_sub1x128_strided<CRIT, true, true><<<grid, dim3(256), 0, st>>>(x, sh, o, th, mode, gam, three, group_rows);
        else k_sub1x128_strided<CRIT, true, false><<<grid, dim3(256), 0, st>>>(x, sh, o, th, mode, gam, three, group_rows);
    } else {
        if (fake) k_sub1x128_strided<CRIT, false, true><<<grid, dim3(256), 0, st>>>(x, sh, o, th, mode, gam, three, group_rows);
        else k_sub1x128_strided<CRIT, false, false><<<grid, dim3(256), 0, st>>>(x, sh, o, th, mode, gam, three, group_rows);
    }
}
static hipError_t launch_sub1x128(const uint16_t* x, const KShape& sh, const KOut& o, int crit, bool defer, float th, uint32_t mode,
                                  const uint32_t* gam, uint32_t three, uint32_t group_rows, hipStream_t st, KProf* prof) {
    ProfScope ps(prof, kKernSub1x128, st);
    const dim3 grid((unsigned)((sh.cols + 127) / 128), (unsigned)clamp_grid_y((sh.rows + 15) / 16));
    if (crit == kCritEq3) launch_sub1x128_crit<kCritEq3>(grid, x, sh, o, defer, th, mode, gam, three, group_rows, st);
    else launch_sub1x128_crit<kCritEq2>(grid, x, sh, o, defer, th, mode, gam, three, group_rows, st);
    return hipGetLastError();
}

// Whether a tile's rows can be addressed through a RowMap; if not, the kernels for padded rows take the operand chunk by chunk.
static bool tensor_rows_fit(const KShape& sh, const KOut& o) {
    const int64_t cpr = sh.cols / 8;
    return cpr < (1 << 28) && row_map_fits(longest_row(sh, o), kTensorChunksPerBlock / cpr + 2);
}
// Fills the chunk layout of a per-tensor operand (or of the amax pass of one): rows of sh.ld elements, outputs as in o.
static void set_tensor_layout(TensorOp& t, const KShape& sh, const KOut& o) {
    const int64_t cpr = sh.cols / 8;
    t.n_chunks = sh.rows * cpr;
    t.n_tiles = (t.n_chunks + kTensorChunksPerBlock - 1) / kTensorChunksPerBlock;
    t.chunks_per_row = cpr;
    t.keep_from = keep_for_second_pass(sh) ? 0 : t.n_tiles;
    t.rm = RowMap{};
    t.rm.ld = sh.ld;
    if (!tensor_rows_fit(sh, o)) return;      // wide: cpr stays 0
    t.rm.cpr = (uint32_t)cpr;
    recip_of(cpr, &t.rm.mul, &t.rm.shift);
    t.rm.step_r = (uint32_t)(256 / cpr);
    t.rm.step_c = (uint32_t)(256 % cpr);
}

// ---- batches ---------------------------------------------------------------------------------
namespace {
constexpr int kStatsMaxWg = 256;
static_assert(kScopeBlocks <= kStatsMaxWg, "a tensor-level decision leaves one statistics record per reduce workgroup");

// Which kernels take an operand.
enum Route {
    kRouteTensorGroup,      // per-tensor: grouped three-pass kernels (dense operands and padded leading dimensions in launches of their own)
    kRouteSubFlat,          // 1 x 128, two types, dense, a whole number of 32-block units: the persistent grouped kernel
    kRouteSubRows,          // 1 x 128, two types, padded leading dimensions or ragged edges: the ROWS form of the same kernel
    kRouteSubGeneral,       // 1 x 128, three types, or rows too long for 32-bit offsets inside a unit
    kRouteTeam,             // 128 x 128, 64 x 64, per-channel rows: a team of lanes keeps the block in registers
    kRouteSubCol,           // 128 x 1
    kRouteChannelCol        // per-channel columns
};
bool item_is_flat(const BatchItem& it) { return is_flat(it.sh, it.o); }
Route route_of(const BatchItem& it) {
    const bool plain = !it.three;
    switch (it.gran) {
    case kGranTensor: return kRouteTensorGroup;
    case kGranSub: {
        const int64_t bpr = (it.sh.cols + 127) / 128;
        if (!plain) return kRouteSubGeneral;
        if (item_is_flat(it) && it.sh.cols % 128 == 0 && (it.sh.rows * bpr) % 32 == 0) return kRouteSubFlat;
        return bpr < (1 << 24) && row_map_fits(longest_row(it.sh, it.o), 32 / bpr + 2) ? kRouteSubRows : kRouteSubGeneral;
    }
    case kGranBlock: case kGranBlock64: case kGranRow: return kRouteTeam;
    case kGranSubCol: return kRouteSubCol;
    default: return kRouteChannelCol;
    }
}
int64_t item_parts(const BatchItem& it) { return geom_parts(make_geom(it.gran, it.sh.rows, it.sh.cols)); }
// A 1 x 128 operand whose blocks are decided one by one can gather its statistics in its own kernel (k_sub1x128_solo_stats)
// when it is alone in its launch and the batch has no per-tensor launch they could ride on.
bool solo_stats_candidate(const BatchItem& it) {
    return it.stats && it.scope == 0 && (route_of(it) == kRouteSubFlat || route_of(it) == kRouteSubRows);
}
constexpr int64_t kStatsOneWg = 4096;        // blocks whose statistics one workgroup of 256 lanes takes
int stats_wgs(int64_t n_part) {                        // riding in a launch of 256-lane workgroups
    if (n_part <= kStatsOneWg) return 1;                // one workgroup writes the result directly
    int64_t w = (n_part + 1023) / 1024;
    return (int)(w > kStatsMaxWg ? kStatsMaxWg : w);
}
int stats_wgs_fast(int64_t n_part) {                   // launch of its own: workgroups of kStatsFastThreads lanes
    if (n_part <= kStatsDirectParts) return 1;
    int64_t w = (n_part + kStatsFastThreads * kStatsFastPerLane - 1) / (kStatsFastThreads * kStatsFastPerLane);
    return (int)(w > kStatsMaxWg ? kStatsMaxWg : w);
}
size_t item_workspace(const BatchItem& it) {
    size_t b = 0;
    if (it.gran == kGranTensor) b += plan_tensor(it.sh.rows, it.sh.cols).bytes;
    else if (it.scope == 1) b += scope_workspace_bytes(item_parts(it));
    if (it.gran == kGranCol) b += column_workspace_bytes(it.sh.rows, it.sh.cols);
    if (it.stats && it.gran != kGranTensor) b += align16(sizeof(StatsRec) * (solo_stats_candidate(it) ? kSubFlatMaxBlocks : kStatsMaxWg));
    if (it.gran != kGranTensor && it.scaling != kScaleFp32) {
        b += 16;                                                                   // group mantissa words (E8M0 uses none; the size stays)
        if (it.scaling == kScaleGam && it.group_rows == 0) b += 2 * align16(sizeof(uint32_t) * kProveMaxWg);   // amax and flush partials of the pre-pass
        if (it.scaling == kScaleGam && it.group_rows != 0) {                       // bands of rows as groups: mantissa table, amax partials
            const size_t n_groups = (size_t)((it.sh.rows + it.group_rows - 1) / it.group_rows);
            b += align16(8 * n_groups) + align16(sizeof(uint32_t) * n_groups * (size_t)band_wgs(it));
        }
    }
    return b;
}
int share(int64_t mine, int64_t total, int budget, int64_t cap) {
    int64_t v = total > 0 ? (mine * budget + total - 1) / total : 1;
    if (v > cap) v = cap;
    if (v > budget) v = budget;
    return (int)(v < 1 ? 1 : v);
}
constexpr int kMaxGroupTensor = 8;
}  // namespace

size_t batch_workspace_bytes(const BatchItem* items, int n) {
    size_t b = 0;
    for (int i = 0; i < n; ++i) b += item_workspace(items[i]);
    return b;
}

namespace {
// What goes along with the passes (see TensorFill), and the statistics that it leaves to the finish pass.
struct StreamFill {
    int form = kFillNone;
    TensorFill table{};
    FillOrder order{};
    SoloStats solo{};
    uint32_t direct = 0u;
};
// One batch call: the launches of every phase, in stream order.  The phases share the workspace cursor, the routes, the
// group-mantissa words of Algorithm 1 and the statistics groups, which is all this object holds.
constexpr int kMaxStatsGroups = (kBatchMax + kMaxGroupStats - 1) / kMaxGroupStats;
struct BatchRun {
    const BatchItem* items;
    int n;
    float near_tol;
    hipStream_t st;
    KProf* prof;
    char* wsp;
    size_t ws_off = 0;
    hipError_t err = hipSuccess;
    Route route[kBatchMax];
    const uint32_t* gam_of[kBatchMax] = {};      // per operand: {mantissa for E4M3, for E5M2, "BF16 proven" flag}
    char* col_ws[kBatchMax] = {};                // per operand with per-channel columns: its column workspace
    GroupStats stats_groups[kMaxStatsGroups];
    int n_stats_groups = 0;
    bool will_ride = false;                      // the batch has grouped per-tensor launches for statistics to ride on
    bool riders_used = false;                    // the first statistics group went along with a per-tensor launch
    bool stats_done[kBatchMax] = {};             // the operand's block kernel has written its statistics already
    int wave_of[kBatchMax] = {};                 // operands that Algorithm 1 reads twice: the group they are taken in; others 0
    int n_waves = 1;
    bool streamed[kBatchMax] = {};               // operands whose two passes have shared a launch: no group (-1)
    bool first_read_keeps[kBatchMax] = {};       // ... and whether the amax pass leaves them in the Infinity Cache

    size_t ws_bytes = 0;
    // Next `bytes` of the caller's workspace.  The phases below carve exactly what item_workspace() adds up; should the
    // two ever drift apart, the call fails (hipErrorOutOfMemory) instead of writing beyond the workspace: once `err`
    // is set no further kernel is launched, so the pointer returned here is never dereferenced.
    char* carve(size_t bytes) {
        const size_t need = align16(bytes);
        if (err != hipSuccess || need > ws_bytes - ws_off) { if (err == hipSuccess) err = hipErrorOutOfMemory; return wsp; }
        char* p = wsp + ws_off;
        ws_off += need;
        return p;
    }
    int fill_strided = -1;                       // the per-tensor launch that takes others along: 0 dense operands, 1 padded rows, -1 none
    int fill_sub = -1, fill_team[kMaxTeamGroup], n_fill_team = 0;
    void plan_fill();
    void make_fill(StreamFill& f, GroupStats& riders, int& ride_final);
    void paired_operands();
    void streamed_operands();
    void assign_waves();
    void group_mantissas(int wave);
    void sub_tensor_operands(int crit, int wave);
    void tensor_level_decisions();
    void collect_statistics();
    void per_tensor_operands(int crit);
    void leftover_statistics();
};

// ---- Algorithm 1, group loop: operands with sub-tensor blocks and GAM / E8M0 scaling get their group
//      mantissas first (GAM: one more read of the operand for its amax)
// Under a tensor-level decision the operands of these granularities gain less from the second read than the launches of every part
// and a slower first pass cost (twelve operands of a layer, us per call in parts of 256 MB; in one go, kept; in one go, not kept):
// per-channel rows 527, 514, 507 (fake quantization 526, 510, 508), 64 x 64 blocks 537, 509, 525 (536, 525, 526), 1 x 128 sub-rows
// with payload 477, 478, 464.  Up to 256 MB they are kept like the others (8192 x 4096 per-channel rows: 51 against 66 us).
bool taken_whole(const BatchItem& it) {
    return scope_proof_applies(it) && (it.gran == kGranRow || it.gran == kGranBlock64 || (it.gran == kGranSub && it.o.fake == nullptr));
}
// The operands of linear layers under the per-channel strategy: rows and columns in common launches (see launch_channel_col_items).
void BatchRun::paired_operands() {
    if (n < 2) return;
    for (int fake = 0; fake < 2 && err == hipSuccess; ++fake) {
        PairRows rows;
        rows.n = 0;
        int row_idx[kPairMax], cols[kPairMax], n_cols = 0;
        bool fits = true;
        for (int i = 0; i < n; ++i) {
            const BatchItem& it = items[i];
            if (it.crit != kCritEq2 || it.three || (it.o.fake != nullptr) != (fake != 0)) continue;
            const bool row = it.gran == kGranRow;
            if (!row && it.gran != kGranCol) continue;
            fits &= row ? rows.n < kPairMax && pair_takes_row(it) : n_cols < kPairMax;
            if (!fits) break;
            if (row) { row_idx[rows.n] = i; rows.ops[rows.n++].it = &it; fits &= it.scaling == rows.ops[0].it->scaling; }
            else cols[n_cols++] = i;
        }
        if (!fits || rows.n == 0 || n_cols == 0 || !columns_pair(items, cols, n_cols)) continue;
        for (int k = 0; k < rows.n; ++k) {
            const int i = row_idx[k];
            rows.ops[k].gam = nullptr; rows.ops[k].sync = nullptr;
            if (items[i].scaling == kScaleGam) {
                gam_of[i] = rows.ops[k].gam = reinterpret_cast<uint32_t*>(carve(16));
                rows.ops[k].sync = reinterpret_cast<uint32_t*>(carve(sizeof(uint32_t) * kStreamWords));
            }
            streamed[i] = true;
        }
        char* ws_of[kPairMax];
        for (int k = 0; k < n_cols; ++k) {
            const int i = cols[k];
            if (items[i].scaling == kScaleGam) gam_of[i] = reinterpret_cast<uint32_t*>(carve(16));
            ws_of[k] = col_ws[i] = carve(column_workspace_bytes(items[i].sh.rows, items[i].sh.cols));
            streamed[i] = true;
        }
        if (err == hipSuccess) err = launch_channel_col_items(items, cols, n_cols, kCritEq2, gam_of, ws_of, &rows, st, prof);
    }
}
// Operands whose two passes share a launch.
void BatchRun::streamed_operands() {
    constexpr int kMost = 12;                    // operands of a launch
    bool beside = false;
    int kind[kBatchMax];
    uint32_t kinds = 0u;
    for (int i = 0; i < n; ++i) {
        const int k = streamed[i] ? -1 : team_stream_kind(items[i]);
        kind[i] = k < 0 ? -1 : 2 * k + (items[i].o.fake != nullptr ? 1 : 0);
        if (k >= 0) kinds |= 1u << kind[i];
        beside |= !streamed[i] && items[i].scaling == kScaleGam && items[i].gran != kGranTensor && items[i].gran != kGranCol && k < 0;
    }
    for (int c = 0; c < 2 * kTeamKinds && err == hipSuccess; ++c) {
        if ((kinds >> c & 1u) == 0u) continue;
        int idx[kBatchMax], cnt = 0;
        for (int i = 0; i < n; ++i)
            if (kind[i] == c) idx[cnt++] = i;
        for (int base = 0; base < cnt && err == hipSuccess; base += kMost) {
            TeamStreamItem ops[kMost];
            const int m = cnt - base < kMost ? cnt - base : kMost;
            int64_t bytes = 0;
            for (int k = 0; k < m; ++k) bytes += items[idx[base + k]].sh.rows * items[idx[base + k]].sh.cols * 2;
            if (!stream_pays(m, bytes, items[idx[base]].gran == kGranBlock, beside)) continue;
            for (int k = 0; k < m; ++k) {
                const int i = idx[base + k];
                ops[k].it = &items[i];
                ops[k].gam = reinterpret_cast<uint32_t*>(carve(16));
                ops[k].sync = reinterpret_cast<uint32_t*>(carve(sizeof(uint32_t) * kStreamWords));
                gam_of[i] = ops[k].gam;
                streamed[i] = true;
            }
            if (err == hipSuccess) err = launch_team_stream_items(ops, m, st, prof);
        }
    }
}
void BatchRun::assign_waves() {
    int64_t bytes = 0, whole_bytes = 0;
    for (int i = 0; i < n; ++i)
        if (streamed[i]) wave_of[i] = -1;
        else if (taken_whole(items[i])) whole_bytes += items[i].sh.rows * items[i].sh.cols * 2;
    const bool whole = whole_bytes > kKeepGroupBytes;
    for (int i = 0; i < n; ++i) {
        const BatchItem& it = items[i];
        first_read_keeps[i] = keep_for_second_pass(it.sh);
        if (streamed[i] || it.gran == kGranTensor || it.gran == kGranCol || it.scaling != kScaleGam) continue;      // (those two group themselves)
        if (whole && taken_whole(it)) continue;
        const int64_t b = it.sh.rows * it.sh.cols * 2;
        if (bytes > 0 && bytes + b > kKeepGroupBytes) { ++n_waves; bytes = 0; }
        bytes += b;
        wave_of[i] = n_waves - 1;
    }
    if (!whole) return;
    if (bytes > 0) ++n_waves;
    for (int i = 0; i < n; ++i)
        if (!streamed[i] && taken_whole(items[i])) {
            wave_of[i] = n_waves - 1;
            first_read_keeps[i] &= items[i].gran == kGranBlock64;
        }
}
void BatchRun::group_mantissas(int wave) {
    int idx[kBatchMax];
    int cnt = 0;
    for (int i = 0; i < n; ++i)
        if (wave_of[i] == wave && items[i].gran != kGranTensor && items[i].scaling == kScaleGam && items[i].group_rows == 0) idx[cnt++] = i;
    // operands whose groups are bands of rows: one mantissa pair per band, in a table behind the four header words
    for (int i = 0; i < n && err == hipSuccess; ++i) {
        const BatchItem& it = items[i];
        if (wave_of[i] != wave || it.group_rows == 0) continue;
        const int64_t n_groups = (it.sh.rows + it.group_rows - 1) / it.group_rows;
        const int wpb = band_wgs(it);
        if (n_groups * wpb > 0x7FFFFFFF) { err = hipErrorInvalidValue; return; }
        uint32_t* gam = reinterpret_cast<uint32_t*>(carve(16 + align16(8 * (size_t)n_groups)));
        uint32_t* part = reinterpret_cast<uint32_t*>(carve(sizeof(uint32_t) * (size_t)n_groups * (size_t)wpb));
        if (err != hipSuccess) return;
        gam_of[i] = gam;
        { ProfScope ps(prof, kKernGroupAmax, st); 
            if (keep_for_second_pass(it.sh)) k_band_amax<true><<<dim3((unsigned)(n_groups * wpb)), dim3(256), 0, st>>>(it.x, it.sh, it.group_rows, wpb, part);
            else k_band_amax<false><<<dim3((unsigned)(n_groups * wpb)), dim3(256), 0, st>>>(it.x, it.sh, it.group_rows, wpb, part); }
        { ProfScope ps(prof, kKernGroupMantissa, st); k_gam_prepare_bands<<<dim3((unsigned)((n_groups + 255) / 256)), dim3(256), 0, st>>>(part, wpb, n_groups, gam, it.o.gmant); }
    }
    // operands whose tensor-level decision the pre-pass may prove: block-shaped pre-pass (group amax and, per block,
    // the elements that are certain to flush), as many operands per launch as its argument table holds
    uint32_t* pv_part[kBatchMax] = {};
    uint32_t* pv_flush[kBatchMax] = {};
    int pv_wg[kBatchMax] = {};
    {
        constexpr int kProveGroup = 12;
        BlockProveItem pv[kProveGroup];
        int pv_item[kProveGroup];
        int n_pv = 0;
        int64_t pv_units = 0;
        auto flush = [&]() {
            if (n_pv == 0 || err != hipSuccess) { n_pv = 0; pv_units = 0; return; }
            for (int j = 0; j < n_pv; ++j) {
                const int64_t units = scope_proof_units(items[pv_item[j]]);
                // twelve operands, 128x128: 0.577 ms per pass at 2048 workgroups in all, 0.564 ms at 4096 and at 8192
                pv[j].n_wg = share(units, pv_units, kProveMaxWg, units);
                pv_wg[pv_item[j]] = pv[j].n_wg;
            }
            ProfScope ps(prof, kKernGroupAmax, st);
            err = launch_block_amax_prove(pv, n_pv, st);
            n_pv = 0; pv_units = 0;
        };
        for (int k = 0; k < cnt && err == hipSuccess; ++k) {
            const int i = idx[k];
            const BatchItem& it = items[i];
            if (!scope_proof_applies(it)) continue;
            pv_part[i] = reinterpret_cast<uint32_t*>(carve(sizeof(uint32_t) * kProveMaxWg));
            pv_flush[i] = reinterpret_cast<uint32_t*>(carve(sizeof(uint32_t) * kProveMaxWg));
            pv[n_pv] = BlockProveItem{it.x, it.sh.rows, it.sh.cols, it.sh.ld, pv_part[i], pv_flush[i], 0, scope_proof_kind(it), first_read_keeps[i] ? 1 : 0};
            pv_units += scope_proof_units(it);
            pv_item[n_pv] = i;
            if (++n_pv == kProveGroup) flush();
        }
        flush();
    }
    for (int base = 0; base < cnt && err == hipSuccess; base += kMaxGroupTensor) {
        const int m = cnt - base < kMaxGroupTensor ? cnt - base : kMaxGroupTensor;
        GroupGam gg; gg.n = m;
        GroupTensor ga[2];                                // dense operands, padded leading dimensions
        int64_t total_tiles[2] = {0, 0};
        int slot_of[kMaxGroupTensor];                     // 2 * slot + layout
        for (int l = 0; l < 2; ++l) { ga[l].n = 0; ga[l].near_tol = near_tol; }
        for (int k = 0; k < m; ++k) {
            const int i = idx[base + k];
            const BatchItem& it = items[i];
            uint32_t* gam = reinterpret_cast<uint32_t*>(carve(16));
            gam_of[i] = gam;
            GamOp& q = gg.op[k];
            q.amax_part = nullptr; q.n_amax = 0; q.mode = (uint32_t)it.scaling; q.gam = gam; q.gmant = it.o.gmant;
            q.flush_part = nullptr; q.flush_need = 0ull; q.skip = 0u;
            slot_of[k] = -1;
            if (it.gran == kGranCol) { q.skip = 1u; continue; }      // the group amax comes out of the column-amax pass
            if (pv_part[i]) {
                q.amax_part = pv_part[i]; q.n_amax = pv_wg[i];
                q.flush_part = pv_flush[i];
                q.flush_need = flush_need_of(it.th, it.sh.rows * it.sh.cols);
                continue;
            }
            uint32_t* part = reinterpret_cast<uint32_t*>(carve(2 * sizeof(uint32_t) * kProveMaxWg));
            q.amax_part = part;
            const int l = it.sh.ld == it.sh.cols ? 0 : 1;
            TensorOp& t = ga[l].op[ga[l].n];
            t = TensorOp{};
            t.x = it.x;
            set_tensor_layout(t, it.sh, KOut{});
            t.amax_part = part;
            total_tiles[l] += t.n_tiles;
            slot_of[k] = 2 * ga[l].n++ + l;
        }
        int a_end[2] = {0, 0};
        for (int l = 0; l < 2; ++l)
            for (int j = 0; j < ga[l].n; ++j) {
                TensorOp& t = ga[l].op[j];
                t.n_amax = share(t.n_tiles, total_tiles[l], total_tiles[l] <= kAmaxOneTile ? kAmaxOneTile : kMaxAmaxBlocks, t.n_tiles);
                a_end[l] += t.n_amax;
                ga[l].amax_end[j] = a_end[l];
            }
        for (int k = 0; k < m; ++k)
            if (slot_of[k] >= 0) gg.op[k].n_amax = ga[slot_of[k] & 1].op[slot_of[k] >> 1].n_amax;
        if (err != hipSuccess) return;
        GroupStats none; none.n = 0; none.near_tol = near_tol;
        if (ga[0].n) {
            ProfScope ps(prof, kKernGroupAmax, st);
            k_tensor_amax_group<false><<<dim3(a_end[0]), dim3(256), 0, st>>>(ga[0], none, a_end[0], 0);
        }
        if (ga[1].n) {
            ProfScope ps(prof, kKernGroupAmax, st);
            k_tensor_amax_group<true><<<dim3(a_end[1]), dim3(256), 0, st>>>(ga[1], none, a_end[1], 0);
        }
        bool any = false;
        for (int k = 0; k < m; ++k) any |= gg.op[k].skip == 0u;
        if (any) { ProfScope ps(prof, kKernGroupMantissa, st); k_gam_prepare<<<dim3(m), dim3(kGamThreads), 0, st>>>(gg); }
    }
}

// Adds an operand to the table of a 1 x 128 launch (all but its running total of units).
template <class G>
void sub_table_add(G& g, const BatchItem& it, const uint32_t* gam) {
    const int k = g.n++;
    const int64_t bpr = (it.sh.cols + 127) / 128;
    g.x[k] = it.x; g.o[k] = it.o; g.th[k] = it.th; g.defer[k] = it.scope == 1;
    g.mode[k] = (uint8_t)it.scaling; g.gam[k] = gam; g.prove[k] = scope_proof_applies(it) ? 1 : 0;
    g.group_rows[k] = (uint32_t)it.group_rows; g.bpr[k] = (uint32_t)bpr;
    g.ld[k] = it.sh.ld; g.cols[k] = it.sh.cols; g.n_part[k] = it.sh.rows * bpr;
    recip_of(bpr < 1 << 24 ? bpr : 1, &g.mul[k], &g.shift[k]);      // (used by the ROWS form only, whose rows are shorter)
}
template <bool ROWS>
void launch_sub_group(const dim3& grid, int crit, bool fake, const GroupSub& g, hipStream_t st) {
    if (fake) {
        if (crit == kCritEq3) k_sub1x128_group<kCritEq3, true, ROWS><<<grid, dim3(256), 0, st>>>(g);
        else k_sub1x128_group<kCritEq2, true, ROWS><<<grid, dim3(256), 0, st>>>(g);
    } else {
        if (crit == kCritEq3) k_sub1x128_group<kCritEq3, false, ROWS><<<grid, dim3(256), 0, st>>>(g);
        else k_sub1x128_group<kCritEq2, false, ROWS><<<grid, dim3(256), 0, st>>>(g);
    }
}
template <bool ROWS>
void launch_solo_stats(const dim3& grid, int crit, bool fake, const SubRiders& one, const SoloStats& ss, hipStream_t st) {
    if (fake) {
        if (crit == kCritEq3) k_sub1x128_solo_stats<kCritEq3, true, ROWS><<<grid, dim3(256), 0, st>>>(one, ss);
        else k_sub1x128_solo_stats<kCritEq2, true, ROWS><<<grid, dim3(256), 0, st>>>(one, ss);
    } else {
        if (crit == kCritEq3) k_sub1x128_solo_stats<kCritEq3, false, ROWS><<<grid, dim3(256), 0, st>>>(one, ss);
        else k_sub1x128_solo_stats<kCritEq2, false, ROWS><<<grid, dim3(256), 0, st>>>(one, ss);
    }
}

// ---- operands with sub-tensor blocks of one criterion
void BatchRun::sub_tensor_operands(int crit, int wave) {
    // ---- small flat 1x128 operands ride on the first 128x128 team launch of the same criterion and output kind
    // (extra workgroups of that launch) instead of paying the ramp and tail of a launch of their own
    TeamRiders riders;
    riders.table.n = 0; riders.blocks = 0; riders.fake = false; riders.used = false;
    int64_t rider_units = 0;
    bool team_has[2] = {false, false};
    for (int i = 0; i < n; ++i)
        if (wave_of[i] == wave && route[i] == kRouteTeam && items[i].crit == crit && team_kind_of(items[i]) == 0) team_has[items[i].o.fake ? 1 : 0] = true;
    // ---- 1x128 sub-channel operands, persistent grouped kernel (FP8 payload, then fake quantization; flat, then ROWS form)
    for (int variant = 0; variant < 4 && err == hipSuccess; ++variant) {
        const bool fake = (variant & 1) != 0, rows_form = (variant & 2) != 0;
        GroupSub g; g.n = 0;
        int64_t total = 0;
        int newest = -1;                                  // the item added to the table last
        auto flush = [&]() {
            if (g.n == 0 || err != hipSuccess) { g.n = 0; total = 0; return; }
            int64_t blocks = (total + 3) / 4;
            const int64_t max_blocks = rows_form ? kSubRowsMaxBlocks : kSubFlatMaxBlocks;
            if (blocks > max_blocks) blocks = max_blocks;
            if (g.n == 1 && !will_ride && solo_stats_candidate(items[newest])) {
                // a lone operand: its kernel gathers the statistics as well
                SoloStats ss;
                ss.rec = reinterpret_cast<StatsRec*>(carve(sizeof(StatsRec) * (size_t)blocks));
                ss.out = static_cast<StatsDev*>(items[newest].stats);
                ss.n_part = item_parts(items[newest]);
                ss.total_elems = (unsigned long long)(items[newest].sh.rows * items[newest].sh.cols);
                ss.edge_missing = (uint32_t)((128 - items[newest].sh.cols % 128) % 128);
                ss.near_tol = near_tol;
                ss.n_rec = (int)blocks;
                if (err != hipSuccess) { g.n = 0; total = 0; return; }
                SubRiders one; one.n = 0;
                sub_table_add(one, items[newest], gam_of[newest]);
                one.unit_end[0] = total;
                {
                    ProfScope ps(prof, kKernSub1x128, st);
                    const dim3 grid((unsigned)blocks);
                    if (rows_form) launch_solo_stats<true>(grid, crit, fake, one, ss, st);
                    else launch_solo_stats<false>(grid, crit, fake, one, ss, st);
                }
                { ProfScope ps2(prof, kKernStatsFinal, st); k_solo_stats_final<<<dim3(1), dim3(kSoloFinalThreads), 0, st>>>(ss); }
                stats_done[newest] = true;
                g.n = 0; total = 0;
                return;
            }
            ProfScope ps(prof, kKernSub1x128, st);
            if (rows_form) launch_sub_group<true>(dim3((unsigned)blocks), crit, fake, g, st);
            else launch_sub_group<false>(dim3((unsigned)blocks), crit, fake, g, st);
            g.n = 0; total = 0;
        };
        for (int i = 0; i < n; ++i) {
            const BatchItem& it = items[i];
            if (wave_of[i] != wave || route[i] != (rows_form ? kRouteSubRows : kRouteSubFlat) || it.crit != crit || (it.o.fake != nullptr) != fake) continue;
            const int64_t n_units = (item_parts(it) + 31) / 32;
            if (!rows_form && n_units <= kSubRiderMaxUnits && team_has[fake] && riders.table.n < kMaxSubRiders &&
                (riders.table.n == 0 || riders.fake == fake)) {
                SubRiders& r = riders.table;
                rider_units += n_units;
                sub_table_add(r, it, gam_of[i]);
                r.unit_end[r.n - 1] = rider_units;
                riders.fake = fake;
                riders.blocks = (rider_units + 3) / 4 < kSubFlatMaxBlocks ? (rider_units + 3) / 4 : kSubFlatMaxBlocks;
            } else {
                total += n_units;
                sub_table_add(g, it, gam_of[i]);
                g.unit_end[g.n - 1] = total;
                newest = i;
                if (g.n == kMaxGroupSub) flush();
            }
        }
        flush();
    }
    // ---- 1x128 sub-channel operands, general kernel
    for (int i = 0; i < n && err == hipSuccess; ++i) {
        const BatchItem& it = items[i];
        if (wave_of[i] != wave || route[i] != kRouteSubGeneral || it.crit != crit) continue;
        err = launch_sub1x128(it.x, it.sh, it.o, crit, it.scope == 1, it.th, (uint32_t)it.scaling, gam_of[i], (uint32_t)it.three,
                              (uint32_t)it.group_rows, st, prof);
    }
    // ---- team kernels: 128x128 and 64x64 blocks, per-channel rows
    for (int kind = 0; kind < kTeamKinds && err == hipSuccess; ++kind) {
        int idx[kBatchMax];
        int cnt = 0;
        for (int i = 0; i < n; ++i)
            if (wave_of[i] == wave && route[i] == kRouteTeam && items[i].crit == crit && team_kind_of(items[i]) == kind) idx[cnt++] = i;
        if (cnt) err = launch_team_items(items, idx, cnt, kind, crit, gam_of, &riders, st, prof);
    }
    if (err == hipSuccess && riders.table.n > 0 && !riders.used) {      // no team launch took them: a launch of their own
        GroupSub g; g.n = riders.table.n;
        for (int k = 0; k < g.n; ++k) {
            const SubRiders& r = riders.table;
            g.unit_end[k] = r.unit_end[k]; g.x[k] = r.x[k]; g.o[k] = r.o[k]; g.th[k] = r.th[k]; g.defer[k] = r.defer[k];
            g.mode[k] = r.mode[k]; g.gam[k] = r.gam[k]; g.prove[k] = r.prove[k]; g.group_rows[k] = r.group_rows[k]; g.bpr[k] = r.bpr[k];
        }
        ProfScope ps(prof, kKernSub1x128, st);
        launch_sub_group<false>(dim3((unsigned)riders.blocks), crit, riders.fake, g, st);
        riders.used = true;
    }
    // ---- 128x1 sub-columns
    if (err == hipSuccess) {
        int idx[kBatchMax];
        int cnt = 0;
        for (int i = 0; i < n; ++i)
            if (wave_of[i] == wave && route[i] == kRouteSubCol && items[i].crit == crit) idx[cnt++] = i;
        if (cnt) err = launch_subcol_items(items, idx, cnt, crit, gam_of, st, prof);
    }
    // ---- per-channel columns
    if (err == hipSuccess) {
        int idx[kBatchMax];
        char* ws_of[kBatchMax];
        int cnt = 0;
        for (int i = 0; i < n; ++i)
            if (wave_of[i] == wave && route[i] == kRouteChannelCol && items[i].crit == crit) {
                ws_of[cnt] = carve(column_workspace_bytes(items[i].sh.rows, items[i].sh.cols));
                col_ws[i] = ws_of[cnt];
                idx[cnt++] = i;
            }
        if (cnt && err == hipSuccess) err = launch_channel_col_items(items, idx, cnt, crit, gam_of, ws_of, nullptr, st, prof);
    }
}

// ---- tensor-level decision (Section 3.1) over the per-block sums the block kernels left behind
void BatchRun::tensor_level_decisions() {
    GroupScope g; g.n = 0;
    int red = 0, copy = 0;
    auto flush = [&]() {
        if (g.n == 0 || err != hipSuccess) { g.n = 0; red = 0; copy = 0; return; }
        bool direct = true;
        for (int k = 0; k < g.n; ++k) direct &= g.op[k].n_part <= (g.op[k].stats ? kScopeDirectStats : kScopeDirect) && g.op[k].col.n_strips == 0;
        if (direct) { ProfScope ps(prof, kKernFallbackCopy, st); k_scope_direct_group<<<dim3(copy), dim3(256), 0, st>>>(g); }
        else {
            { ProfScope ps(prof, kKernScopeReduce, st); k_scope_reduce_group<<<dim3(red), dim3(256), 0, st>>>(g); }
            { ProfScope ps(prof, kKernFallbackCopy, st); k_scope_copy_group<<<dim3(copy), dim3(256), 0, st>>>(g); }
        }
        g.n = 0; red = 0; copy = 0;
    };
    int64_t total_elems = 0, unproven_bytes = 0;
    int n_unproven = 0;                                    // operands whose BF16 payload, if any, is left to the copy launch
    for (int i = 0; i < n; ++i) {
        const BatchItem& it = items[i];
        if (it.gran == kGranTensor || it.scope != 1) continue;
        total_elems += it.sh.rows * it.sh.cols;
        if (it.o.bf16 == nullptr || scope_proof_applies(it) || column_tensor_proof_applies(it)) continue;
        ++n_unproven;
        unproven_bytes += it.sh.rows * it.sh.cols * 2;
    }
    const int budget = scope_copy_budget(n_unproven, unproven_bytes);
    for (int i = 0; i < n; ++i) {
        const BatchItem& it = items[i];
        if (it.gran == kGranTensor || it.scope != 1) continue;
        ScopeOp& t = g.op[g.n];
        char* w = carve(scope_workspace_bytes(0));
        t.err_sum = it.o.err_sum; t.err5_sum = it.o.err5_sum; t.nnz = it.o.nnz; t.mask = it.o.mask;
        t.n_part = item_parts(it);
        t.part_err = reinterpret_cast<double*>(w); t.part_err5 = t.part_err + kScopeBlocks;
        t.part_nnz = reinterpret_cast<unsigned long long*>(w) + 2 * kScopeBlocks;
        t.decision = reinterpret_cast<uint32_t*>(w + 3 * sizeof(double) * kScopeBlocks);
        t.th = it.th; t.crit = it.crit;
        t.proven = scope_proof_applies(it) ? gam_of[i] + 2 : nullptr;
        if (column_tensor_proof_applies(it)) t.proven = column_tensor_proven_word(col_ws[i], it.sh.rows, it.sh.cols);
        t.col = ColumnSums{};
        if (it.gran == kGranCol) t.col = column_sums_of(col_ws[i], it.sh.rows, it.sh.cols, it.o.amax);
        int64_t want = t.col.n_strips ? (t.n_part + 255) / 256 : (t.n_part + 1023) / 1024;      // (a column is a sum over the strips)
        t.n_red = (int)(want < 1 ? 1 : (want > kScopeBlocks ? kScopeBlocks : want));
        t.stats = static_cast<StatsDev*>(it.stats);
        t.rec = it.stats ? reinterpret_cast<StatsRec*>(carve(sizeof(StatsRec) * kStatsMaxWg)) : nullptr;
        t.near_tol = near_tol;
        stats_done[i] = true;
        t.x = it.x; t.bf16 = it.o.bf16;
        t.rows = it.sh.rows; t.cols = it.sh.cols; t.ld = it.sh.ld; t.ld_bf16 = it.o.ld_bf16;
        red += t.n_red;
        {   // workgroups of the decision / mask / copy launch: enough for the copy, and never fewer than the reduce pass had
            const int c = it.o.bf16 ? share(it.sh.rows * it.sh.cols, total_elems, budget, budget) : 1;
            copy += c > t.n_red ? c : t.n_red;
        }
        g.red_end[g.n] = red; g.copy_end[g.n] = copy;
        if (++g.n == kMaxGroupScope) flush();
    }
    flush();
}

// ---- statistics of the operands with sub-tensor blocks: their kernels (and tensor-level decisions) are done, so the
//      first group can ride on the first per-tensor launches: partial records in the shadow of pass A, the combine
//      step next to the finish pass.  Groups that find no such launch run on their own at the end.
void BatchRun::collect_statistics() {
    GroupStats* g = nullptr;
    for (int i = 0; i < n; ++i) {
        const BatchItem& it = items[i];
        if (!it.stats || it.gran == kGranTensor || stats_done[i]) continue;
        if (!g || g->n == kMaxGroupStats) { g = &stats_groups[n_stats_groups++]; g->n = 0; g->near_tol = near_tol; }
        StatsOp& t = g->op[g->n];
        t.err_sum = it.o.err_sum; t.nnz = it.o.nnz; t.mask = it.o.mask;
        t.geom = make_geom(it.gran, it.sh.rows, it.sh.cols);
        t.n_part = geom_parts(t.geom);
        t.th = it.th;
        t.rec = reinterpret_cast<StatsRec*>(carve(sizeof(StatsRec) * kStatsMaxWg));
        t.out = static_cast<StatsDev*>(it.stats);
        // the first group rides on the first grouped per-tensor launches if the batch has any, the others are launched on their own
        const bool rides = n_stats_groups == 1 && will_ride;
        g->wg_end[g->n] = (g->n ? g->wg_end[g->n - 1] : 0) + (rides ? stats_wgs(t.n_part) : stats_wgs_fast(t.n_part));
        ++g->n;
    }
}

// The launches of a table of per-tensor operands: pass A and pass B over one part of the table after the other (see
// kKeepGroupBytes), then one finish pass for all.  Statistics of sub-tensor operands ride in extra workgroups of the first and
// the last one.
struct TensorPart {
    int a0, a1, s0, s1;      // workgroups of pass A and pass B
    int lds;                 // residency cap
};
// Both passes in one launch, under Eq. 2 with two types.  us per call, with a launch for each pass / streamed: the six gradients of a layer (and its
// other operands, statistics) 8192 tokens x hidden 4096 409 / 382.5, 4096 x 3072 236 / 212, 1024 x 2048 107 / 97, 512 x 1024 47 / 37; six of 4096 x 4096
// kept in E4M3 102 / 81, two 38 / 35; three of 1024 x 4096 (768 tiles, a workgroup each in either pass) 21.6 / 23.5, four 24.3 / 24.8, six 36.4 / 32.0.  Alone
// there is nothing to overlap: dense 4096 x 4096 23.0 / 24.2, 4099 x 5000 48.7 / 46.4 (with a 1 x 128 operand), 8192 x 4096 36.8 / 35.8, 14336 x 4096 53.5 /
// 55.1, 8192 x 14336 97.7 / 100.5 (falling back to BF16 135 / 132.6); padded rows 4096 x 4096 24.3 / 25.5, 4099 x 5000 31.1 / 28.4, 8192 x 4096
// 40.4 / 39.2, 8192 x 14336 105.6 / 106.2 (140.9 / 133.2).
bool tensor_stream_pays(int n, int64_t tiles, bool strided, bool ride) {
    if (n == 1) return tiles > 1024 && (strided || tiles <= 2560);
    return tiles > (ride ? kAmaxOneTile : 1280);
}
template <bool STRIDED>
hipError_t launch_tensor_stream(GroupTensor& g, const GroupStats& riders, int ride_partial, int c_end, int ride_final, bool fake, int polls, StreamFill& fill,
                                hipStream_t st, KProf* prof) {
    if (fill.form != kFillNone && (fake || (STRIDED && fill.form == kFillFlat))) return hipErrorInvalidValue;      // not instantiated below
    StreamClear clear;
    clear.n = g.n;
    uint32_t groups = 0u, largest = 0u;
    int slots = 0, most = 0;
    for (int k = 0; k < g.n; ++k) {
        TensorOp& t = g.op[k];
        const int tiles = (int)t.n_tiles;
        const uint32_t mine = stream_groups(tiles);
        groups += mine;
        slots += (tiles + 7) / 8 * 8;
        g.amax_end[k] = (int32_t)groups;
        g.slot_end[k] = slots;
        t.n_slots = tiles;
        clear.tiles[k] = tiles;
        clear.words[k] = reinterpret_cast<uint32_t*>(t.err5);
        if (g.n > 1) t.keep_from = 0;                     // the second pass follows at the distance of one operand
        if (mine > largest) largest = mine;
        if (tiles > most) most = tiles;
    }
    StreamOrder order;
    if (!stream_order(order, groups, largest, (uint32_t)slots / 8u)) return hipErrorInvalidValue;
    if (fill.form != kFillNone) {
        FillOrder& f = fill.order;
        // The 1 x 128 operand, whose workgroups take longer than the others', goes in early: behind the first pass of a lone per-tensor operand, while
        // that is collected, beside the first passes of several.  us per call, behind / beside: 1000 x 4096 and a slice like it 16.8 / 18.3, 4099 x 5000
        // 47.8 / 50.0, 8192 x 14336 206 / 224; a layer of 8192 x hidden 4096 376.5 / 373.6, 1 x 128 and three gradients of 4096 x 4096 62.7 / 61.6.
        const uint32_t span = g.n == 1 ? 0u : order.lead, rest = groups + (uint32_t)slots / 8u - order.lead + f.team.n;
        f.alone = order.lead - span;
        f.early = span + f.sub.n;
        if (!make_spread(f.sub, f.sub.n, f.early) || !make_spread(f.team, f.team.n, rest)) return hipErrorInvalidValue;
    }
    {
        ProfScope ps(prof, kKernStreamClear, st);
        k_tensor_stream_clear<<<dim3(stream_clear_wgs(most), (unsigned)g.n + (fill.form != kFillNone ? 1u : 0u)), dim3(256), 0, st>>>(clear, fill.table);
    }
    {
        ProfScope ps(prof, kKernTensorStream, st);
        const FillOrder& fo = fill.order;
        const dim3 grid(((unsigned)ride_partial + 7u) / 8u * 8u + 8u * groups + (unsigned)slots + (fill.form != kFillNone ? 8u * (fo.sub.n + fo.team.n) : 0u));
        // (gradients of a layer 383.0 us per call uncapped, 382.5 at 5, 382.1 at 4, 382.4 at 3 workgroups per compute unit, kept lean 347.5, 347.7, 346.2,
        // 354.9; a slice of 4099 x 5000 28.6, 28.6, 30.1, 28.5)
        if (fake) k_tensor_stream<true, STRIDED, kFillNone><<<grid, dim3(256), kResidency5, st>>>(g, riders, order, ride_partial, polls, fo);
        else if (fill.form == kFillNone) k_tensor_stream<false, STRIDED, kFillNone><<<grid, dim3(256), kResidency5, st>>>(g, riders, order, ride_partial, polls, fo);
        else if (STRIDED || fill.form == kFillRows) k_tensor_stream<false, STRIDED, kFillRows><<<grid, dim3(256), kResidency5, st>>>(g, riders, order, ride_partial, polls, fo);
        else k_tensor_stream<false, false, kFillFlat><<<grid, dim3(256), kResidency5, st>>>(g, riders, order, ride_partial, polls, fo);
    }
    ProfScope ps(prof, kKernFallbackCopy, st);
    if (fill.form != kFillNone) k_tensor_finish_fill<STRIDED><<<dim3(c_end + ride_final), dim3(256), 0, st>>>(g, riders, c_end, fill.direct, fill.solo);
    else k_tensor_finish_group<kCritEq2, STRIDED><<<dim3(c_end + ride_final), dim3(256), 0, st>>>(g, riders, c_end);
    return hipGetLastError();
}
template <bool STRIDED>
void launch_tensor_passes(const GroupTensor& g, const TensorPart* parts, int n_parts, const GroupStats& riders, int ride_partial, int c_end,
                          int ride_final, int crit, bool fake, hipStream_t st, KProf* prof) {
    for (int k = 0; k < n_parts; ++k) {
        const TensorPart& p = parts[k];
        const int ride = k == 0 ? ride_partial : 0;
        {
            ProfScope ps(prof, kKernTensorAmax, st);
            k_tensor_amax_group<STRIDED><<<dim3(p.a1 - p.a0 + ride), dim3(256), 0, st>>>(g, riders, p.a1 - p.a0, p.a0);
        }
        ProfScope ps(prof, kKernTensorQuant, st);
        const dim3 grid(p.s1 - p.s0);
        if (fake) {
            if (crit == kCritEq3) k_tensor_quant_group<kCritEq3, true, STRIDED><<<grid, dim3(256), p.lds, st>>>(g, p.s0);
            else k_tensor_quant_group<kCritEq2, true, STRIDED><<<grid, dim3(256), p.lds, st>>>(g, p.s0);
        } else {
            if (crit == kCritEq3) k_tensor_quant_group<kCritEq3, false, STRIDED><<<grid, dim3(256), p.lds, st>>>(g, p.s0);
            else k_tensor_quant_group<kCritEq2, false, STRIDED><<<grid, dim3(256), p.lds, st>>>(g, p.s0);
        }
    }
    {
        ProfScope ps(prof, kKernFallbackCopy, st);
        if (crit == kCritEq3) k_tensor_finish_group<kCritEq3, STRIDED><<<dim3(c_end + ride_final), dim3(256), 0, st>>>(g, riders, c_end);
        else k_tensor_finish_group<kCritEq2, STRIDED><<<dim3(c_end + ride_final), dim3(256), 0, st>>>(g, riders, c_end);
    }
}
// A small operand that is alone: two launches from a table of one operand.  Such a call is a chain of launches, so what counts is their
// number, what the host spends on each (3.8 KB of kernel arguments for a table of eight operands and the statistics' riders, 0.4 KB
// here) and the depth of a workgroup's work.  The workgroups wait to be told, so at most half of those that the registers let be
// resident together are launched.
// us per call, here / with the three launches that larger operands take: dense, kept in E4M3, 64 x 256 9.4 / 13.8, 1024 x 1024
// 11.1 / 14.1, 1024 x 4096 11.9 / 15.5, 2048 x 4096 14.6 / 18.4; kept in BF16 without a proof (Eq. 3) 1024 x 1024 12.7 / 15.9, 1024 x 4096
// 13.4 / 18.4; padded rows 256 x 4096 9.9 / 11.5, 2048 x 4096 17.1 / 18.8.  (4096 x 4096, beyond: three launches, 23.1.)
constexpr int64_t one_max_chunks(int crit) { return crit == kCritEq3 ? 1 << 19 : 1 << 20; }      // (Eq. 3 with eight chunks per lane does not fit the registers)
constexpr int64_t kOnePadded2 = 1 << 18, kOneShared = 1 << 19;
constexpr int kDenseAmaxLanes = 512;      // us per call at 256 / 512 / 1024 lanes: 64 x 256 9.5 / 9.2 / 9.4, 1024 x 1024 11.2 / 11.2 / 11.4, 2048 x 4096 14.8 / 14.6 / 14.9
static_assert(one_max_chunks(kCritEq2) <= (int64_t)kAmaxOneTile * kTensorChunksPerBlock, "a workgroup per dense tile");
static_assert(kOnePadded2 <= (int64_t)kOneMaxSlots * 512 && kOneShared <= (int64_t)kOneMaxSlots * 1024 && one_max_chunks(kCritEq2) <= (int64_t)kOneMaxSlots * 2048,
              "a slot per tile");
struct OneShape {
    int lanes, chunks;
};
// Padded rows, two chunks per lane up to kOneShared: with 256 x 4 above kOnePadded2 the ordinary path takes the same time (768 x 4096 12.2 us
// both), but one that goes chunk by chunk, a chain of latencies per lane, takes longer than with three launches: rows too long for a
// RowMap (1 x 4 194 296) 19.9 us with two chunks, 24.1 with four, 20.5 with three launches; 768 x 4096 with an infinity, Eq. 3, 20.6, 24.3, 22.0.
OneShape one_shape(int64_t n_chunks, bool dense) {
    if (n_chunks > kOneShared) return {256, 8};
    if (dense) return {512, 4};
    if (n_chunks <= kOnePadded2) return {256, 2};
    return {512, 2};
}
template <int CRIT, bool FAKE>
void launch_one_quant(const OneTensor& o, const OneShape& s, int slots, int polls, hipStream_t st) {
    const dim3 grid(slots), block(s.lanes);
    if (s.lanes == 512 && s.chunks == 4) k_tensor_quant_one<CRIT, FAKE, 512, 4><<<grid, block, 0, st>>>(o, polls);
    else if (s.lanes == 512) k_tensor_quant_one<CRIT, FAKE, 512, 2><<<grid, block, 0, st>>>(o, polls);
    else if (s.chunks == 2) k_tensor_quant_one<CRIT, FAKE, 256, 2><<<grid, block, 0, st>>>(o, polls);
    else if constexpr (CRIT == kCritEq2) k_tensor_quant_one<CRIT, FAKE, 256, 8><<<grid, block, 0, st>>>(o, polls);
}
void launch_one_tensor(const TensorOp& t, float near_tol, int crit, bool fake, int polls, hipStream_t st, KProf* prof) {
    OneTensor o;
    o.n = 1; o.near_tol = near_tol; o.op[0] = t;
    const bool dense = (t.flags & kTensorDense) != 0u;
    const OneShape s = one_shape(t.n_chunks, dense);
    const int slots = (int)((t.n_chunks + s.lanes * s.chunks - 1) / (s.lanes * s.chunks));
    TensorOp& a = o.op[0];
    const int amax_tile = dense ? kTensorChunksPerBlock : 256 * kSmallChunksPerThread;
    a.n_tiles = (a.n_chunks + amax_tile - 1) / amax_tile;      // pass A's tiles
    a.n_amax = (int)(a.n_tiles < kAmaxOneTile ? a.n_tiles : kAmaxOneTile);
    a.keep_from = 0;
    a.n_slots = slots;
    o.amax_end[0] = a.n_amax; o.slot_end[0] = slots; o.copy_end[0] = 0;
    {
        ProfScope ps(prof, kKernTensorAmax, st);
        if (dense) k_tensor_amax_one_dense<kDenseAmaxLanes, kTensorChunksPerBlock / kDenseAmaxLanes><<<dim3(a.n_amax), dim3(kDenseAmaxLanes), 0, st>>>(o);
        else k_tensor_amax_one<<<dim3(a.n_amax), dim3(256), 0, st>>>(o);
    }
    a.n_tiles = slots;
    ProfScope ps(prof, kKernTensorQuant, st);
    if (fake) {
        if (crit == kCritEq3) launch_one_quant<kCritEq3, true>(o, s, slots, polls, st);
        else launch_one_quant<kCritEq2, true>(o, s, slots, polls, st);
    } else {
        if (crit == kCritEq3) launch_one_quant<kCritEq3, false>(o, s, slots, polls, st);
        else launch_one_quant<kCritEq2, false>(o, s, slots, polls, st);
    }
}
// Can the operand's two passes share a launch?
bool tensor_streams(const BatchItem& it) {
    if (it.gran != kGranTensor || it.crit != kCritEq2 || it.three) return false;
    if ((it.sh.rows * (it.sh.cols / 8) + kTensorChunksPerBlock - 1) / kTensorChunksPerBlock > kTensorStreamMaxTiles) return false;
    return item_is_flat(it) || tensor_rows_fit(it.sh, it.o);
}
// A small per-tensor operand alone has kernels of its own, whose two launches a 1 x 128 operand or blocks beside it do not outweigh unless they bring
// statistics.  us per call apart / together, without: slices of 64 x 1024 12.7 / 14.2, 512 x 2048 12.8 / 15.2; 2000 x 4096 kept in E4M3 with a 1 x 128 operand
// of 1000 x 4096 19.1 / 20.3, falling back without a proof 22.6 / 25.1, with one 20.8 / 19.8, in padded rows beside 64 x 4096 18.3 / 19.9, 20.4 / 26.1, 18.7 /
// 18.3; beyond (see one_max_chunks) 4096 x 4096 27.1 / 24.5, 2500 x 5000 37.2 / 33.0.  With statistics 18.5 / 14.5, 19.1 / 15.3,
// 1000 x 4096 22.8 / 16.8, 2500 x 5000 37.9 / 32.7, 4099 x 5000 48.2 / 47.8, 8192 x 4096 66.2 / 62.3.  Layers with statistics: 8192 tokens x hidden 4096 382.9 / 373.6 (lean,
// without 347.2 / 328.9), 4096 x 2048 107.5 / 102.1, 512 x 1024 37.1 / 33.6, 64 x 256 21.3 / 16.1.
bool takes_two_launches(const BatchItem& it) {
    return it.sh.rows * (it.sh.cols / 8) <= one_max_chunks(it.crit) && (!item_is_flat(it) || tensor_rows_fit(it.sh, it.o));
}
// Which operands go along with the passes of per-tensor ones (see TensorFill): those decided block by block under Eq. 2 with two types, FP8
// payload and no pre-pass, of which one may have 1 x 128 blocks; with statistics, up to what one workgroup counts of 128 x 128 blocks.
void BatchRun::plan_fill() {
    if (n < 2) return;
    for (int strided = 0; strided < 2 && fill_strided < 0; ++strided) {
        int cnt = 0;
        int64_t tiles = 0, pass_groups = 0;                // (groups of eight workgroups, see TensorFill)
        bool all = true, small = false;                    // (`small`: of the last, where it is alone)
        for (int i = 0; i < n; ++i) {
            const BatchItem& it = items[i];
            if (it.gran != kGranTensor || it.crit != kCritEq2 || it.o.fake || item_is_flat(it) != (strided == 0)) continue;
            all &= tensor_streams(it);
            small = takes_two_launches(it);
            ++cnt;
            const int64_t own = (it.sh.rows * (it.sh.cols / 8) + kTensorChunksPerBlock - 1) / kTensorChunksPerBlock;
            tiles += own;
            pass_groups += 2 * ((own + 7) / 8) + 1;
        }
        bool counts = false;                               // the call counts statistics (those of a per-tensor operand come with its decision)
        for (int i = 0; i < n; ++i) counts |= items[i].stats != nullptr && items[i].gran != kGranTensor;
        if (cnt == 0 || cnt > kMaxGroupTensor || !all || (cnt == 1 && !counts && small)) continue;
        int others = 0, counted = 0;                       // statistics of operands that do not go along, of blocks that do
        int subs = 0, subs_counted = 0;
        int64_t team_wgs = 0;
        bool launch_stays = false;                         // of 128 x 128 blocks, for other operands
        // Blocks beyond what the launch's order can be divided into (some 370 000, 12 GB) keep a launch of their own.
        auto spread = [&](int64_t wgs) { return spread_fits((uint64_t)(wgs + 7) / 8, (uint64_t)(pass_groups + (wgs + 7) / 8)); };
        for (int i = 0; i < n; ++i) {
            const BatchItem& it = items[i];
            if (it.gran == kGranTensor) continue;
            const Route own = route_of(it);
            const bool plain = it.crit == kCritEq2 && it.scope == 0 && !it.three && !it.o.fake && it.scaling != kScaleGam;
            if (plain && (own == kRouteSubFlat || own == kRouteSubRows)) {
                ++subs;
                subs_counted += it.stats != nullptr;
                if (!strided || own == kRouteSubRows) fill_sub = i;
            }
            else if (plain && own == kRouteTeam && team_kind_of(it) == kTeamWg128 && !team_needs_edge(it, kTeamWg128) && n_fill_team < kMaxTeamGroup &&
                     (!it.stats || item_parts(it) <= kStatsOneWg) && spread(team_wgs + item_parts(it))) {
                fill_team[n_fill_team++] = i;
                team_wgs += item_parts(it);
                counted += it.stats != nullptr;
            } else {
                others += it.stats != nullptr;
                launch_stays |= own == kRouteTeam && wave_of[i] == 0 && it.crit == kCritEq2 && !it.o.fake && team_kind_of(it) == kTeamWg128 && !team_needs_edge(it, kTeamWg128);
            }
        }
        if (subs > 1) fill_sub = -1;
        if (fill_sub < 0) others += subs_counted;          // (the one that goes along leaves records of its own)
        // Blocks alone save nothing where their launch stays for others: then the passes have to pay by themselves, or be of several operands beside many
        // blocks.  us per call apart / together, beside blocks of 2304 x 384 under GAM scales: one of 3681 x 1336 with blocks of 2048 x 4096 26.7 / 31.1,
        // 8192 x 4096 39.5 / 41.6; that and 2059 x 1760 with 2048 x 4096 32.0 / 33.2, 4096 x 4096 37.7 / 36.8, 8192 x 4096 45.2 / 44.0 (where no launch
        // stays 1408 x 1280 23.8 / 20.4).
        const bool pays = fill_sub >= 0 || !launch_stays || (cnt > 1 && team_wgs >= 1024) || tensor_stream_pays(cnt, tiles, strided != 0, others > 0);
        if ((fill_sub < 0 && n_fill_team == 0) || !pays || others + counted > kMaxGroupStats) { fill_sub = -1; n_fill_team = 0; continue; }
        fill_strided = strided;
    }
    if (fill_strided < 0) return;
    if (fill_sub >= 0) { wave_of[fill_sub] = -1; stats_done[fill_sub] = true; }
    for (int k = 0; k < n_fill_team; ++k) { wave_of[fill_team[k]] = -1; stats_done[fill_team[k]] = true; }
}
void BatchRun::make_fill(StreamFill& f, GroupStats& riders, int& ride_final) {
    TensorFill& t = f.table;
    f.form = fill_strided ? kFillRows : kFillFlat;      // (beside padded rows only the rows form exists; without a 1 x 128 operand nothing runs it)
    int64_t units = 0;
    t.team.n = n_fill_team;
    for (int k = 0; k < n_fill_team; ++k) {
        const BatchItem& it = items[fill_team[k]];
        int64_t units_x;
        units += team_units(it, kTeamWg128, units_x);
        set_team_op(t.team.op[k], it, units_x, nullptr);
        t.team.unit_end[k] = units;
        if (!it.stats) continue;
        if (riders.n == kMaxGroupStats) { err = hipErrorInvalidValue; return; }      // (not where plan_fill has counted right)
        StatsOp& s = riders.op[riders.n];
        s.err_sum = it.o.err_sum; s.nnz = it.o.nnz; s.mask = it.o.mask;
        s.geom = make_geom(it.gran, it.sh.rows, it.sh.cols);
        s.n_part = geom_parts(s.geom);
        s.th = it.th; s.rec = nullptr; s.out = static_cast<StatsDev*>(it.stats);
        riders.wg_end[riders.n] = (riders.n ? riders.wg_end[riders.n - 1] : 0) + 1;
        f.direct |= 1u << riders.n++;
    }
    ride_final = riders.n;
    if (fill_sub >= 0) {
        const BatchItem& it = items[fill_sub];
        if (route_of(it) == kRouteSubRows) f.form = kFillRows;
        t.sub.n = 0;
        sub_table_add(t.sub, it, nullptr);
        t.sub.unit_end[0] = (item_parts(it) + 31) / 32;
        int64_t per = (t.sub.unit_end[0] + 4 * kSubFlatMaxBlocks - 1) / (4 * kSubFlatMaxBlocks);
        t.sub_blocks = (int32_t)((t.sub.unit_end[0] + 4 * per - 1) / (4 * per));
        t.near_tol = near_tol;
        if (it.stats) {
            t.sub_rec = reinterpret_cast<StatsRec*>(carve(sizeof(StatsRec) * (size_t)t.sub_blocks));
            f.solo.rec = t.sub_rec; f.solo.out = static_cast<StatsDev*>(it.stats);
            f.solo.n_part = item_parts(it);
            f.solo.total_elems = (unsigned long long)(it.sh.rows * it.sh.cols);
            f.solo.edge_missing = (uint32_t)((128 - it.sh.cols % 128) % 128);
            f.solo.near_tol = near_tol;
            f.solo.n_rec = t.sub_blocks;
            ++ride_final;
        }
    }
    f.order.sub.n = (uint32_t)(t.sub_blocks + 7) / 8u;
    f.order.team.n = (uint32_t)((units + 7) / 8);
}
void BatchRun::per_tensor_operands(int crit) {
    // ---- per-tensor operands: amax pass, quantize pass, finish (+ fallback copy) pass; FP8 payload and fake
    //      quantization are different kernels, and so are dense operands and padded leading dimensions
    for (int variant = 0; variant < 4 && err == hipSuccess; ++variant) {
        const bool fake = (variant & 1) != 0, strided = (variant & 2) != 0;
        int idx[kMaxGroupTensor];
        int cnt = 0;
        auto flush = [&]() {
            if (cnt == 0 || err != hipSuccess) { cnt = 0; return; }
            GroupTensor g; g.n = cnt; g.near_tol = near_tol;
            const bool ride = !riders_used && n_stats_groups > 0;
            const BatchItem& it0 = items[idx[0]];
            // (the kernels of the two launches address rows through a RowMap, so a dense operand whose rows are too long for it stays with the
            // dense kernels, which number chunks without it: 1 x 8 388 608 kept in BF16 45.2 us as one of these, without a proof, 17.6 with the dense kernels)
            const bool filled = fill_strided == (strided ? 1 : 0) && crit == kCritEq2 && !fake;
            const bool one = cnt == 1 && !ride && !filled && takes_two_launches(it0);
            int64_t all_tiles = 0;
            for (int k = 0; k < cnt; ++k) {
                const BatchItem& it = items[idx[k]];
                TensorOp& t = g.op[k];
                t.x = it.x; t.o = it.o; t.th = it.th; t.mode = (uint32_t)it.scaling; t.three = it.three ? 1u : 0u;
                t.flags = strided ? 0u : kTensorDense | kTensorReport | (it.lean ? kTensorLean : 0u);      // (padded rows always get their payload, and report no proof)
                set_tensor_layout(t, it.sh, it.o);
                all_tiles += t.n_tiles;
                const TensorPlan pl = plan_tensor(it.sh.rows, it.sh.cols);
                char* w = carve(pl.bytes);
                t.amax_part = reinterpret_cast<uint32_t*>(w + pl.off_amax_part);
                t.err = reinterpret_cast<float*>(w + pl.off_err_part);
                t.err5 = reinterpret_cast<float*>(w + pl.off_err5_part);
                t.zero = reinterpret_cast<uint32_t*>(w + pl.off_nnz_part);
                t.abits = reinterpret_cast<uint32_t*>(w + pl.off_decision);
                t.flush_part = reinterpret_cast<uint32_t*>(w + pl.off_flush_part);
                t.flush_need = 0ull;
                if (crit == kCritEq2 && it.o.bf16 && !it.three && it.th > 0.0f && it.th < 0.9f)
                    t.flush_need = flush_need_of(it.th, it.sh.rows * it.sh.cols);
                t.stats = static_cast<StatsDev*>(it.stats);
            }
            if (err != hipSuccess) { cnt = 0; return; }      // the workspace ran out while carving
            TensorPart parts[kMaxGroupTensor];
            int n_parts = 0, a_end = 0, s_end = 0, c_end = 0;
            for (int first = 0; first < cnt;) {
                int64_t bytes = 0, total_tiles = 0;
                int last = first;                            // operands first .. last - 1 form a part
                for (; last < cnt; ++last) {
                    const BatchItem& it = items[idx[last]];
                    const int64_t b = it.sh.rows * it.sh.cols * 2;
                    if (last > first && bytes + b > kKeepGroupBytes) break;
                    bytes += b;
                    total_tiles += g.op[last].n_tiles;
                }
                // Launch shape.  Several operands in the launch: one 32 KB tile per workgroup of pass B (up to 16384), at most
                // three workgroups resident per compute unit.  One operand alone does better with persistent workgroups that are
                // all resident from the start (224 MiB kept in E4M3: 97.6 us per call with 512 workgroups in pass A and 1280 in pass B, 99.9
                // with 768 and 1536, 102.9 with one tile per workgroup of pass B; falling back to BF16 134.8, 136.0 and 134.6; a
                // layer with its six gradients 408 us, 414 at 768 and 1536).
                const bool solo = last - first == 1 && total_tiles <= 2000ll * kSoloQuantBlocks;
                // Up to kAmaxOneTile tiles, and what fits the chip at once in pass B, a workgroup takes one tile.
                const int amax_cap = total_tiles <= kAmaxOneTile ? kAmaxOneTile : kMaxAmaxBlocks;
                const int quant_cap = !solo ? kMaxQuantBlocks : (total_tiles <= kQuantOneTile ? kQuantOneTile : kSoloQuantBlocks);
                TensorPart& p = parts[n_parts++];
                p.lds = solo ? 0 : kResidency3;
                p.a0 = a_end; p.s0 = s_end;
                for (int k = first; k < last; ++k) {
                    TensorOp& t = g.op[k];
                    t.n_amax = share(t.n_tiles, total_tiles, amax_cap, t.n_tiles);
                    t.n_slots = share(t.n_tiles, total_tiles, quant_cap, t.n_tiles);
                    t.keep_from = bytes > kKeepTensorBytes ? t.n_tiles - t.n_tiles * (kKeepTensorBytes >> 15) / total_tiles : 0;
                    a_end += t.n_amax; s_end += t.n_slots;
                    c_end += (t.o.bf16 || t.three) ? share(t.n_tiles, all_tiles, 2048, 2048) : 1;
                    g.amax_end[k] = a_end; g.slot_end[k] = s_end; g.copy_end[k] = c_end;
                }
                p.a1 = a_end; p.s1 = s_end;
                first = last;
            }
            GroupStats riders; riders.n = 0; riders.near_tol = near_tol;
            int ride_partial = 0, ride_final = 0;
            if (ride) {
                riders = stats_groups[0];
                ride_partial = riders.wg_end[riders.n - 1];
                ride_final = ride_partial > riders.n ? riders.n : 0;      // single-workgroup operands are final already
                riders_used = true;
            }
            bool stream = filled || (crit == kCritEq2 && tensor_stream_pays(cnt, all_tiles, strided, ride));
            for (int k = 0; k < cnt; ++k) stream &= tensor_streams(items[idx[k]]);
            if (!one && stream) {
                StreamFill fill;
                if (filled) {
                    make_fill(fill, riders, ride_final);
                    if (err != hipSuccess) { cnt = 0; return; }
                }
                err = strided ? launch_tensor_stream<true>(g, riders, ride_partial, c_end, ride_final, fake, it0.polls, fill, st, prof)
                              : launch_tensor_stream<false>(g, riders, ride_partial, c_end, ride_final, fake, it0.polls, fill, st, prof);
            }
            else if (one) launch_one_tensor(g.op[0], near_tol, crit, fake, it0.polls, st, prof);
            else if (strided) launch_tensor_passes<true>(g, parts, n_parts, riders, ride_partial, c_end, ride_final, crit, fake, st, prof);
            else launch_tensor_passes<false>(g, parts, n_parts, riders, ride_partial, c_end, ride_final, crit, fake, st, prof);
            cnt = 0;
        };
        for (int i = 0; i < n; ++i) {
            const BatchItem& it = items[i];
            if (route[i] != kRouteTensorGroup || it.crit != crit || (it.o.fake != nullptr) != fake || item_is_flat(it) == strided) continue;
            const int64_t n_tiles = (it.sh.rows * it.sh.cols / 8 + kTensorChunksPerBlock - 1) / kTensorChunksPerBlock;
            if (n_tiles > kMaxTensorTiles) { err = hipErrorInvalidValue; return; }
            idx[cnt] = i;
            if (++cnt == kMaxGroupTensor) flush();
        }
        flush();
    }
}

// ---- statistics of the operands with sub-tensor blocks that found no per-tensor launch to ride on
void BatchRun::leftover_statistics() {
    for (int k = riders_used ? 1 : 0; k < n_stats_groups && err == hipSuccess; ++k) {
        const GroupStats& g = stats_groups[k];
        const int wg_total = g.wg_end[g.n - 1];
        { ProfScope ps(prof, kKernStatsPartial, st); k_stats_group_partial<<<dim3(wg_total), dim3(kStatsFastThreads), 0, st>>>(g); }
        if (wg_total > g.n) { ProfScope ps(prof, kKernStatsFinal, st); k_stats_group_final<<<dim3(g.n), dim3(256), 0, st>>>(g); }
    }
}

}  // namespace

hipError_t launch_batch(const BatchItem* items, int n, float near_tol, void* ws, size_t ws_bytes, hipStream_t st, KProf* prof) {
    static_assert(sizeof(GroupSub) <= 3800 && sizeof(GroupTensor) + sizeof(GroupStats) <= 3800 &&
                  sizeof(GroupGam) <= 3800 && sizeof(GroupScope) <= 3800, "kernel-argument segment is 4 KB");
    static_assert(sizeof(StatsRec) == 128, "StatsRec layout");
    BatchRun run;
    run.items = items; run.n = n; run.near_tol = near_tol; run.st = st; run.prof = prof;
    run.wsp = static_cast<char*>(ws);
    run.ws_bytes = ws_bytes;
    for (int i = 0; i < n; ++i) run.route[i] = route_of(items[i]);
    {   // A single 1 x 128 operand that needs the ROWS form gets it from kSubRowsAlone blocks on: a wave works through 32 blocks
        // there, which a small operand alone pays as latency, but several operands share the launch.
        int rows_form = 0, last = 0;
        for (int i = 0; i < n; ++i)
            if (run.route[i] == kRouteSubRows) { ++rows_form; last = i; }
        if (rows_form == 1 && item_parts(items[last]) < kSubRowsAlone) run.route[last] = kRouteSubGeneral;
    }
    for (int i = 0; i < n; ++i) run.will_ride |= run.route[i] == kRouteTensorGroup;
    run.paired_operands();
    run.streamed_operands();
    run.assign_waves();
    run.plan_fill();
    for (int wave = 0; wave < run.n_waves && run.err == hipSuccess; ++wave) {
        run.group_mantissas(wave);
        for (int crit = 0; crit < 2 && run.err == hipSuccess; ++crit) run.sub_tensor_operands(crit, wave);
    }
    if (run.err == hipSuccess) run.tensor_level_decisions();
    // the statistics of the sub-tensor operands are collected after their kernels (and tensor-level decisions)
    if (run.err == hipSuccess) run.collect_statistics();
    for (int crit = 0; crit < 2 && run.err == hipSuccess; ++crit) run.per_tensor_operands(crit);
    run.leftover_statistics();
    if (run.err != hipSuccess) return run.err;
    return hipGetLastError();
}

hipError_t launch_dequantize_batch(const DeqItem* items, int n, hipStream_t st) {
    static_assert(sizeof(GroupDeq) <= 3800, "kernel-argument segment is 4 KB");
    GroupDeq g; g.n = 0;
    int64_t total = 0;
    auto flush = [&]() {
        if (g.n == 0) return;
        k_dequant_group<<<dim3((unsigned)total), dim3(256), 0, st>>>(g);
        g.n = 0; total = 0;
    };
    for (int i = 0; i < n; ++i) {
        const DeqItem& it = items[i];
        const StatsGeom& geom = it.geom;
        const int prl = block_shift(geom.pr, geom.rows, 64), pcl = block_shift(geom.pc, geom.cols, 64);
        if (geom.pc == 1 && geom.cols > 1) {       // one column per block: its own kernel
            const dim3 grid((unsigned)((geom.cols + 127) / 128), (unsigned)clamp_grid_y((geom.rows + 127) / 128));
            k_dequant_columns<<<grid, dim3(256), 0, st>>>(geom, prl, it.fp8, it.ld_fp8, it.scale, it.mask, it.bf16, it.ld_bf16, it.y, it.ld_y,
                                                          it.e8m0, it.gmant, it.group_rows);
            continue;
        }
        TensorOp layout;
        KOut o{};
        o.fake = it.y; o.ld_fake = it.ld_y;
        if (it.bf16) { o.bf16 = const_cast<uint16_t*>(it.bf16); o.ld_bf16 = it.ld_bf16; }
        set_tensor_layout(layout, KShape{geom.rows, geom.cols, it.ld_fp8}, o);
        layout.n_tiles = (layout.n_chunks + 256 * kDeqChunks - 1) / (256 * kDeqChunks);
        if (layout.rm.cpr == 0u || layout.n_tiles > 0x7FFFFFFF || it.group_rows > 0x7FFFFFFF) {      // 64-bit addresses, one chunk at a time
            const dim3 grid((unsigned)((geom.cols + 127) / 128), (unsigned)clamp_grid_y((geom.rows + 15) / 16));
            k_dequant<<<grid, dim3(256), 0, st>>>(geom, prl, pcl, it.fp8, it.ld_fp8, it.scale, it.mask, it.bf16, it.ld_bf16, it.y, it.ld_y, it.e8m0,
                                                  it.gmant, it.group_rows);
            continue;
        }
        if (total + layout.n_tiles > 0x7FFFFFFF) flush();
        DeqOp& t = g.op[g.n];
        t.rm = layout.rm; t.n_chunks = layout.n_chunks; t.gc = geom.gc; t.pr_log2 = prl; t.pc_log2 = block_shift(geom.pc, geom.cols, 32);
        t.fp8 = it.fp8; t.scale = it.scale; t.mask = it.mask; t.bf16 = it.bf16; t.y = it.y; t.e8m0 = it.e8m0; t.gmant = it.gmant;
        t.ld_fp8 = (uint32_t)it.ld_fp8; t.ld_bf16 = (uint32_t)it.ld_bf16; t.ld_y = (uint32_t)it.ld_y;
        t.group_rows = (uint32_t)it.group_rows;
        recip_of(it.group_rows ? it.group_rows : 1, &t.group_mul, &t.group_shift);
        total += layout.n_tiles;
        g.tile_end[g.n] = (int32_t)total;
        if (++g.n == kMaxGroupDeq) flush();
    }
    flush();
    return hipGetLastError();
}

hipError_t launch_select_stats(const StatsGeom& geom, const float* err_sum, const uint32_t* nnz,
                               const uint8_t* mask, float th, float near_tol, void* out_dev, hipStream_t st) {
    static_assert(sizeof(StatsDev) == 144, "mor_stats layout");
    StatsDev* sd = static_cast<StatsDev*>(out_dev);
    const int64_t n_part = geom_parts(geom);
    if (n_part <= 8192) {
        k_stats_single<<<dim3(1), dim3(256), 0, st>>>(n_part, geom, err_sum, nnz, mask, th, near_tol, sd);
    } else {
        k_stats_zero<<<dim3(1), dim3(64), 0, st>>>(sd);
        int64_t want = (n_part + 1023) / 1024;
        const int nb = (int)(want > 1024 ? 1024 : want);
        k_stats_multi<<<dim3(nb), dim3(256), 0, st>>>(n_part, geom, err_sum, nnz, mask, th, near_tol, sd);
        k_stats_finish<<<dim3(1), dim3(64), 0, st>>>(n_part, (unsigned long long)(geom.rows * geom.cols), sd);
    }
    return hipGetLastError();
}

hipError_t launch_histogram_update(uint32_t* hist, const void* stats_dev, int clear, hipStream_t st) {
    k_histogram_update<<<dim3(1), dim3(64), 0, st>>>(hist, static_cast<const StatsDev*>(stats_dev), clear);
    return hipGetLastError();
}

}  // namespace mor
