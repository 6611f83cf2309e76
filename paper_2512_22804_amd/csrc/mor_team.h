// "Team" kernels' body: a team of threads (a wave or a whole workgroup) owns one block and keeps it in registers, so one HBM pass
// computes amax, scale, codes, error sums and the decision.
#pragma once

#include <type_traits>

#include "mor_device.h"
#include "mor_launch.h"
#include "mor_stream.h"

namespace mor {

constexpr int kChunks = 8;     // 16-byte chunks per lane

// ======================================================================================
// Team kernels
// ======================================================================================
enum {
    kTeamWg128 = 0,     // 128 x 128 block, one workgroup
    kTeamHalf64 = 1,    // 64 x 64 blocks, two side by side per wave (32 lanes each, 16 chunks per lane), so that a wave's loads
                        // cover 256-byte row segments; a workgroup takes a tile of 128 rows x 256 columns (eight blocks)
    kTeamWaveRow = 2,   // one row of at most 4096 elements, one wave; four rows per workgroup
    kTeamWgRow = 3,     // one row of at most 16384 elements, one workgroup of 256
    kTeamBigRow = 4     // one row of at most 65536 elements, one workgroup of 1024
};
constexpr int kWaveRowCols = 64 * 8 * kChunks;      // longest row that a wave holds
static_assert(kTeamBigRow + 1 == kTeamKinds, "the batch launcher walks over every team kind");
constexpr int kMaxTeamGroup = 12;
struct TeamOp {
    const uint16_t* x;
    KOut o;
    int64_t ld, rows, cols;
    int64_t units_x;        // 128-column tiles per row of tiles (block kinds)
    float th;
    uint8_t defer, mode, three, prove;      // prove: gam[2] != 0 says the tensor-level BF16 decision is already proven
    uint32_t group_rows;                    // GAM with bands of rows as groups (0: one group)
    const uint32_t* gam;
};
struct GroupTeam {
    int n;
    int64_t unit_end[kMaxTeamGroup];
    TeamOp op[kMaxTeamGroup];
};
struct TeamShared {
    uint32_t u[16];
    float f[32];
};

template <int TEAM> __device__ __forceinline__ constexpr bool team_is_wg() { return TEAM == kTeamWg128 || TEAM == kTeamWgRow || TEAM == kTeamBigRow; }
template <int TEAM> __device__ __forceinline__ constexpr int team_threads() { return TEAM == kTeamBigRow ? 1024 : 256; }
template <int TEAM> __device__ __forceinline__ constexpr int team_waves() { return team_threads<TEAM>() / 64; }
template <int TEAM> __device__ __forceinline__ constexpr int team_chunks() { return TEAM == kTeamHalf64 ? 16 : kChunks; }

// All-reduce over the 32 lanes of a half-wave team: lanes with the same bit 3 (8-lane groups of the four 16-lane rows).
// The lanes of the other half never enter, so the two blocks of a wave may sit in different branches.
__device__ __forceinline__ uint32_t half_allmax_u32(uint32_t v) {
    v = max(v, dpp_u32<kDppXor1>(v));
    v = max(v, dpp_u32<kDppXor2>(v));
    v = max(v, dpp_u32<kDppHalfMirror>(v));
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = max(r[0], r[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return max(q[0], q[1]);
}
__device__ __forceinline__ uint32_t half_allsum_u32(uint32_t v) {
    v += dpp_u32<kDppXor1>(v);
    v += dpp_u32<kDppXor2>(v);
    v += dpp_u32<kDppHalfMirror>(v);
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = r[0] + r[1];
    const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return q[0] + q[1];
}
__device__ __forceinline__ float half_allsum_f32(float v) {
    v += dpp_f32<kDppXor1>(v);
    v += dpp_f32<kDppXor2>(v);
    v += dpp_f32<kDppHalfMirror>(v);
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

// All-reduce over the team.  Workgroup teams combine the four wave results through LDS (every thread
// of the workgroup must call); wave teams stay inside the wave.
template <int TEAM>
__device__ __forceinline__ uint32_t team_allmax(uint32_t v, TeamShared& sh) {
    if constexpr (TEAM == kTeamHalf64) return half_allmax_u32(v);
    v = wave_allmax_u32(v);
    if constexpr (team_is_wg<TEAM>()) {
        if ((threadIdx.x & 63) == 0) sh.u[threadIdx.x >> 6] = v;
        __syncthreads();
        v = sh.u[0];
#pragma unroll
        for (int k = 1; k < team_waves<TEAM>(); ++k) v = max(v, sh.u[k]);
        __syncthreads();
    }
    return v;
}
// `b` (the E5M2 error sum) is only reduced when WITH_B; otherwise it stays as it is (zero under Eq. 2).
template <int TEAM, bool WITH_B>
__device__ __forceinline__ void team_allsum3(float& a, float& b, uint32_t& z, TeamShared& sh) {
    if constexpr (TEAM == kTeamHalf64) {
        a = half_allsum_f32(a);
        if constexpr (WITH_B) b = half_allsum_f32(b);
        z = half_allsum_u32(z);
        return;
    }
    a = wave_allsum_f32(a);
    if constexpr (WITH_B) b = wave_allsum_f32(b);
    z = wave_allsum_u32(z);
    if constexpr (team_is_wg<TEAM>()) {
        constexpr int NW = team_waves<TEAM>();
        const int w = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) { sh.f[w] = a; if constexpr (WITH_B) sh.f[NW + w] = b; sh.u[w] = z; }
        __syncthreads();
        a = 0.0f; z = 0u;
        if constexpr (WITH_B) b = 0.0f;
#pragma unroll
        for (int k = 0; k < NW; k += 4) {       // fixed order: deterministic
            a += (sh.f[k] + sh.f[k + 1]) + (sh.f[k + 2] + sh.f[k + 3]);
            if constexpr (WITH_B) b += (sh.f[NW + k] + sh.f[NW + k + 1]) + (sh.f[NW + k + 2] + sh.f[NW + k + 3]);
            z += (sh.u[k] + sh.u[k + 1]) + (sh.u[k + 2] + sh.u[k + 3]);
        }
        __syncthreads();
    }
}

// An operand whose pre-pass shares the launch (see mor_stream.h).
struct StreamUnit {
    const uint32_t* told;      // the copy to look at
    int polls;
};
enum { kTeamAlone = 0,         // the operand's figures come from earlier launches
       kTeamStream = 1,        // from the first pass in this launch; `scan` finds them out from the operand itself
       kTeamTold = 2 };        // from the first pass in an earlier launch

// EDGE = false: the operand has no partial blocks (block teams), or its rows are a whole number of the
// team's sweeps (row teams), so chunk validity is uniform over the team and costs no per-lane predicates.
template <int TEAM, int CRIT, bool FAKE, bool EDGE, int FROM, class Scan>
__device__ __forceinline__ void team_block(const TeamOp& t, int64_t unit, TeamShared& sh, const StreamUnit& su, Scan scan) {
    constexpr bool PIPE = FROM != kTeamAlone;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const KOut& o = t.o;
    // ---- geometry: block index p, origin (r0, c0), valid extent h x wd, this lane's chunk positions
    constexpr int NCH = team_chunks<TEAM>();
    int64_t p, r0, c0;
    int h, wd, trow, tcol, rstep, cstep;
    int bcol = 0;                                          // kTeamHalf64: this lane's column inside its block
    bool active = true, leader;
    if constexpr (TEAM == kTeamWg128) {
        const int64_t tr = unit / t.units_x, tc = unit - tr * t.units_x;
        p = unit; r0 = tr * 128; c0 = tc * 128;
        trow = tid >> 4; tcol = (tid & 15) * 8; rstep = 16; cstep = 0;
        h = (int)(t.rows - r0 < 128 ? t.rows - r0 : 128); wd = (int)(t.cols - c0 < 128 ? t.cols - c0 : 128);
        leader = tid == 0;
    } else if constexpr (TEAM == kTeamHalf64) {
        // wave w: rows (w >> 1) * 64 .., columns (w & 1) * 128 .. of the workgroup's 128 x 256 tile; lanes with bit 3 set
        // own the right one of the wave's two blocks
        const int64_t tr = unit / t.units_x, tc = unit - tr * t.units_x;
        const int64_t gc = (t.cols + 63) / 64;
        const int side = (lane >> 3) & 1;
        r0 = tr * 128 + (w >> 1) * 64; c0 = tc * 256 + (w & 1) * 128;
        if (r0 >= t.rows || c0 >= t.cols) return;          // the whole wave is outside: uniform, and no barrier follows
        p = (r0 >> 6) * gc + (c0 >> 6) + side;
        trow = lane >> 4; tcol = (lane & 15) * 8; rstep = 4; cstep = 0;
        bcol = tcol & 63;
        h = (int)(t.rows - r0 < 64 ? t.rows - r0 : 64);
        const int64_t left = t.cols - (c0 + side * 64);
        wd = (int)(left < 0 ? 0 : (left < 64 ? left : 64));   // 0: this lane's block lies outside the tensor
        leader = (lane & 0x37) == 0 && wd > 0;
    } else if constexpr (TEAM == kTeamWaveRow) {
        p = unit * 4 + w; r0 = p; c0 = 0;
        active = p < t.rows;
        trow = 0; tcol = lane * 8; rstep = 0; cstep = 64 * 8;
        h = 1; wd = (int)t.cols;
        leader = lane == 0;
    } else {
        p = unit; r0 = p; c0 = 0;
        trow = 0; tcol = tid * 8; rstep = 0; cstep = team_threads<TEAM>() * 8;
        h = 1; wd = (int)t.cols;
        leader = tid == 0;
    }
    if (!active) return;                                   // wave teams only: no barrier is skipped
    const uint16_t* __restrict__ src = t.x + (r0 + trow) * t.ld + c0 + tcol;
    const int64_t src_step = (int64_t)rstep * t.ld + cstep;
    // Whole-block operands of the block teams use plain pointers; everything else (ragged edges, rows) goes through
    // bounds-checked buffer accesses relative to the block origin, where a lane outside the block costs no branch.
    constexpr bool BUF = EDGE || TEAM == kTeamWaveRow || TEAM == kTeamWgRow || TEAM == kTeamBigRow;
    auto in_block = [&](int i) -> bool {
        if constexpr (TEAM == kTeamHalf64) return (trow + i * rstep < h) && (bcol < wd);
        else return (trow + i * rstep < h) && (tcol + i * cstep < wd);
    };
    auto is_valid = [&](int i) -> bool {
        if constexpr (BUF) return in_block(i);
        else return true;
    };
    const BufRsrc rx = make_buf(t.x + r0 * t.ld + c0);
    const uint32_t xoff = (uint32_t)((trow * t.ld + tcol) * 2), xstep = (uint32_t)(src_step * 2);
    uint32_t told = 0u;
    if constexpr (PIPE) told = agent_load(su.told);      // (before the block's loads, so that it is there before them)
    u32x4 raw[NCH];
    auto load_block = [&](uint32_t off) {
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            if constexpr (BUF || PIPE) raw[i] = buf_load16(rx, is_valid(i) ? off : kBufOutside, i * xstep);
            else raw[i] = load16(src + i * src_step);
        }
    };
    load_block(xoff);
    if constexpr (FROM == kTeamTold) told = (uint32_t)__builtin_amdgcn_readfirstlane((int)told);
    if constexpr (FROM == kTeamStream) {
        // The first pass ends well before the launch comes to the operand's blocks, so this is a look and no wait.
        told = stream_told(su.told, told, su.polls);
        if (__builtin_expect(told == 0u, 0)) {
            told = scan();
            uint32_t off = xoff;
            asm volatile("" : "+v"(off));                  // the block is loaded again, so that its registers need not be kept meanwhile
            load_block(off);
        }
    }
    // ---- amax and zero count (chunks outside the tensor count as zeros and change nothing)
    Scan8 sc{0u, 0u};
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        scan8(raw[i], sc);
        if constexpr (PIPE) asm volatile("" : "+v"(sc.amax2), "+v"(sc.zero2));      // (else the zero count follows the amax, with all masked words kept for it: 133 registers at 64 x 64 instead of 101)
    }
    // pin both results here: otherwise the compiler sinks the zero count below the quantization sweep and keeps the
    // 32 masked words of the block alive across it
    asm volatile("" : "+v"(sc.amax2), "+v"(sc.zero2));
    const uint32_t abits = team_allmax<TEAM>(fold_max16(sc.amax2), sh);
    const uint32_t mode = PIPE ? (uint32_t)kScaleGam : (uint32_t)t.mode;
    uint32_t mg = 0u, mg5 = 0u;
    if constexpr (PIPE) mg = group_mantissa_bits(told & kAmaxBits, kE4M3Max, kScaleGam);
    else if (mode == kScaleGam) { const uint32_t* gw = gam_words(t.gam, t.group_rows, r0); mg = gw[0]; mg5 = gw[1]; }
    float s = block_scale(abits, kE4M3Max, mode, mg);
    float s5 = 0.0f;                                       // only Eq. 3 and the three-way recipe look at E5M2
    if (!PIPE && (CRIT == kCritEq3 || t.three)) s5 = block_scale(abits, kE5M2Max, mode, mg5);
    // ---- destinations
    uint8_t* __restrict__ dst8 = FAKE ? nullptr : o.fp8 + (r0 + trow) * o.ld_fp8 + c0 + tcol;
    const int64_t dst8_step = (int64_t)rstep * o.ld_fp8 + cstep;
    uint16_t* __restrict__ dstf = FAKE ? o.fake + (r0 + trow) * o.ld_fake + c0 + tcol : nullptr;
    const int64_t dstf_step = (int64_t)rstep * o.ld_fake + cstep;
    const BufRsrc r8 = make_buf(FAKE ? nullptr : o.fp8 + r0 * o.ld_fp8 + c0);
    const uint32_t off8 = (uint32_t)(trow * o.ld_fp8 + tcol), step8 = (uint32_t)dst8_step;
    const BufRsrc rf = make_buf(FAKE ? o.fake + r0 * o.ld_fake + c0 : nullptr);
    const uint32_t offf = (uint32_t)((trow * o.ld_fake + tcol) * 2), stepf = (uint32_t)(dstf_step * 2);
    const bool fast = abits < fast_amax_limit(mode);
    // quantizes the block with scale `sc_` for format E5M2 ? E5M2 : E4M3; returns this lane's error sum
    auto quantize = [&](auto fmt, float sc_, bool emit) -> float {
        constexpr bool E5 = decltype(fmt)::value;
        const float s_inv = FAKE ? 1.0f / sc_ : 0.0f;        // correctly rounded IEEE division
        float e0 = 0.0f, e1 = 0.0f;
        if (fast) {
#pragma unroll
            for (int i = 0; i < NCH; ++i) {
                u32x4 deq;
                const u32x2 codes = quant8_fast_deq<E5, FAKE>(raw[i], sc_, s_inv, e0, e1, deq);
                // (fake quantization always stores through the buffer window: `emit` is a run-time value there, and a
                // branch around the stores would split the sweep into basic blocks and cost > 100 registers)
                if constexpr (BUF || FAKE) {
                    const bool put = emit && is_valid(i);
                    if constexpr (FAKE) buf_store16(rf, put ? offf + i * stepf : kBufOutside, deq);
                    else buf_store8(r8, put ? off8 : kBufOutside, i * step8, codes);
                } else if (emit) {
                    if constexpr (FAKE) store16(dstf + i * dstf_step, deq);
                    else store8(dst8 + i * dst8_step, codes);
                }
                __builtin_amdgcn_sched_barrier(0);            // one chunk at a time keeps the register count down
            }
        } else {
#pragma clang loop unroll(disable)
            for (int i = 0; i < NCH; ++i)
                if (in_block(i))
                    e0 += quant8_careful_mem<E5>(src + i * src_step, sc_, emit && !FAKE ? dst8 + i * dst8_step : nullptr,
                                                 emit && FAKE ? dstf + i * dstf_step : nullptr, s_inv);
        }
        return e0 + e1;
    };
    // tensor-level decision already proven by the pre-pass (uniform): the BF16 payload is stored below; a fake-quantized
    // output of such an operand is its input, so the de-quantized values are not stored at all
    bool proven = false;
    if constexpr (PIPE) proven = (told & kToldProven) != 0u;
    else if (t.prove) proven = t.gam[2] != 0u;
    float err, err5 = 0.0f;
    if (CRIT == kCritEq3 && fast && s5 == 128.0f * s) {
        // both formats in one sweep, one reciprocal per element (see quant8_dual)
        const float s_inv = FAKE ? 1.0f / s : 0.0f;
        float e0 = 0.0f, e1 = 0.0f, f0 = 0.0f, f1 = 0.0f;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            u32x4 deq;
            const u32x2 codes = quant8_dual<FAKE>(raw[i], s, s_inv, e0, e1, f0, f1, deq);
            if constexpr (BUF) {
                if constexpr (FAKE) buf_store16(rf, is_valid(i) ? offf + i * stepf : kBufOutside, deq);
                else buf_store8(r8, is_valid(i) ? off8 : kBufOutside, i * step8, codes);
            } else {
                if constexpr (FAKE) store16(dstf + i * dstf_step, deq);
                else store8(dst8 + i * dst8_step, codes);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        err = e0 + e1;
        err5 = f0 + f1;
    } else {
        err = quantize(std::false_type{}, s, !(FAKE && proven));
        if constexpr (CRIT == kCritEq3) err5 = quantize(std::true_type{}, s5, false);
    }
    uint32_t zeros = fold_add16(sc.zero2);
    team_allsum3<TEAM, CRIT == kCritEq3>(err, err5, zeros, sh);
    constexpr uint32_t kTeamElems = (team_is_wg<TEAM>() ? (uint32_t)team_threads<TEAM>() : (TEAM == kTeamHalf64 ? 32u : 64u)) * NCH * 8u;
    const uint32_t nnz = kTeamElems - zeros;
    if (abits >= kInfBits) { err = __builtin_inff(); err5 = __builtin_inff(); }
    const bool defer = t.defer != 0;
    uint32_t mask = defer ? 0u : ((CRIT == kCritEq3) ? decide_eq3(err, err5) : decide_eq2(err, nnz, t.th));
    // ---- three-way recipe: a block that failed M_1 is kept in E5M2 if its dynamic range fits (Eq. 4)
    uint32_t amin_bits = 0u;
    if (!PIPE && t.three && mask == 1u) {                  // uniform over the team
        uint32_t mn2 = 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            u32x4 w = raw[i];
            asm volatile("" : "+v"(w.x), "+v"(w.y), "+v"(w.z), "+v"(w.w));      // no reuse of the masked words of the amax sweep
            mn2 = min_nonzero_m1(w, mn2);
        }
        const uint32_t mn = ~team_allmax<TEAM>(~fold_min16(mn2), sh) & 0xFFFFu;
        amin_bits = nnz ? mn + 1u : 0u;
        if (range_fits_e5m2(abits, amin_bits, nnz)) {
            mask = 2u;
            s = s5;
            (void)quantize(std::true_type{}, s5, true);    // the E5M2 payload replaces the E4M3 one
        }
    }
    if (leader) {
        o.scale[p] = s;
        o.amax[p] = __uint_as_float(abits << 16);
        o.err_sum[p] = err;
        o.nnz[p] = nnz;
        if constexpr (CRIT == kCritEq3) o.err5_sum[p] = err5;
        if (!defer) o.mask[p] = (uint8_t)mask;
        if (mode != kScaleFp32 && o.e8m0) o.e8m0[p] = (uint8_t)(__float_as_uint(s) >> 23);
        if (mode == kScaleE8M0 && p == 0) zero_group_mantissa(o.gmant);
        if (!PIPE && t.three && o.amin) o.amin[p] = __uint_as_float(amin_bits << 16);
    }
    const bool keep = mask == 1u || proven;                // (a deferred decision has mask 0 here)
    if (keep && o.bf16) {                                  // BF16: the block stays as it is
        uint16_t* __restrict__ dbf = o.bf16 + (r0 + trow) * o.ld_bf16 + c0 + tcol;
        const int64_t dbf_step = (int64_t)rstep * o.ld_bf16 + cstep;
        const BufRsrc rb = make_buf(o.bf16 + r0 * o.ld_bf16 + c0);
        const uint32_t offb = (uint32_t)((trow * o.ld_bf16 + tcol) * 2), stepb = (uint32_t)(dbf_step * 2);
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            if constexpr (BUF) buf_store16(rb, is_valid(i) ? offb + i * stepb : kBufOutside, raw[i]);
            else store16(dbf + i * dbf_step, raw[i]);
        }
    }
}

// Does the operand need per-lane validity predicates in the team kernel of this kind?
inline bool team_needs_edge(const BatchItem& it, int kind) {
    switch (kind) {
    case kTeamWg128: return it.sh.rows % 128 != 0 || it.sh.cols % 128 != 0;
    case kTeamHalf64: return it.sh.rows % 64 != 0 || it.sh.cols % 128 != 0;      // a wave spans 128 columns
    default: return false;      // row teams always use the bounds-checked accesses
    }
}
inline int64_t team_units(const BatchItem& it, int kind, int64_t& units_x) {
    units_x = kind == kTeamHalf64 ? (it.sh.cols + 255) / 256 : (it.sh.cols + 127) / 128;
    if (kind == kTeamWg128 || kind == kTeamHalf64) return ((it.sh.rows + 127) / 128) * units_x;
    return kind == kTeamWaveRow ? (it.sh.rows + 3) / 4 : it.sh.rows;
}
inline void set_team_op(TeamOp& u, const BatchItem& it, int64_t units_x, const uint32_t* gam) {
    u.x = it.x; u.o = it.o; u.ld = it.sh.ld; u.rows = it.sh.rows; u.cols = it.sh.cols;
    u.units_x = units_x;
    u.th = it.th; u.defer = it.scope == 1; u.mode = (uint8_t)it.scaling; u.three = (uint8_t)it.three;
    u.prove = scope_proof_applies(it);
    u.gam = gam;
    u.group_rows = (uint32_t)it.group_rows;
}

}  // namespace mor
