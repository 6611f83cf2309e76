// Operands that are read twice (amax first, then quantize), both passes over several of them in ONE launch.
//
// The launch walks over the operands' tiles twice at once: the first pass (amax, elements certain to flush) leads, the blocks follow at a
// distance of the largest operand and some more, so that what they read again lies in the Infinity Cache, and reads and writes are mixed
// evenly all the way.  A workgroup of the first pass leaves its figures in a word of its own; one workgroup behind an operand's last tile
// collects them and tells the blocks' workgroups.  Workgroups are dispatched in order, so what one waits for has as a rule started before; but
// the XCDs start their shares each by itself, and one that other work holds up can lag behind those that wait already.  So no wait is
// without end: who is not told in time takes the figures together itself, counting the tiles that are missing (see stream_scan).
// Against one launch per pass over parts of 256 MB: a boundary between launches costs some 5 us (the last workgroups of one, the first
// loads of the next), and a pass that only reads leaves the writes to the other.  Bare passes over 960 MB, 2 bytes read, then 2 read and
// 2 written per element: 448 us in parts, 417 with one part's first pass beside the other's second, of 2 + 3 written 518 and 492.
#pragma once

#include "mor_device.h"
#include "mor_launch.h"

namespace mor {

// The operand's words in the workspace: copies of what is told, a line each, then a word for each tile of the first pass.
constexpr int kToldLine = 32, kToldCopies = 32;
constexpr int kStreamTiles = kToldCopies * kToldLine;
constexpr int kStreamMaxTiles = kStreamWords - kStreamTiles;
// A tile's word: bit 31 (it is there), its certain flushes (16384 at most), its amax pattern.  What is told: bit 31, bit 30 (the BF16
// decision is proven), the operand's amax pattern.
constexpr uint32_t kThere = 0x80000000u, kToldProven = 0x40000000u, kAmaxBits = 0x7FFFu;
constexpr int kFlushShift = 15;

// Order of the launch, in groups of eight workgroups (one for each XCD): `lead` groups of the first pass, `mixed` groups of which
// mixed_first belong to the first pass, the remaining blocks.
struct StreamOrder {
    uint32_t lead, mixed, mixed_first, mul, shift;      // (reciprocal of `mixed`)
};
struct StreamPlace {
    bool first;
    uint32_t group;          // among those of its kind
};
__device__ __forceinline__ StreamPlace stream_place(const StreamOrder& o, uint32_t group) {
    if (group < o.lead) return {true, group};
    const uint32_t m = group - o.lead;
    if (m >= o.mixed) return {false, m - o.mixed_first};
    const uint32_t before = recip_div(m * o.mixed_first, o.mul, o.shift);
    const bool first = recip_div((m + 1u) * o.mixed_first, o.mul, o.shift) != before;
    return {first, first ? o.lead + before : m - before};
}
// Groups of the first pass between an operand's last tile and its first block, at least, some 10 us: layer of twelve operands at 128 x 128,
// fake quantization, 64 431.1, 128 430.5, 192 433.6, 256 434.8 us per call.
constexpr uint32_t kStreamMargin = 128;
inline bool stream_order(StreamOrder& o, uint32_t first_groups, uint32_t largest, uint32_t block_groups) {
    o.lead = largest + kStreamMargin;
    if (o.lead > first_groups) o.lead = first_groups;
    o.mixed_first = first_groups - o.lead;
    o.mixed = o.mixed_first + (uint32_t)((uint64_t)block_groups * o.mixed_first / first_groups);
    o.mul = o.shift = 0u;
    if ((uint64_t)(o.mixed + 1) * o.mixed_first >= 0x7FFFFFFFull) return false;
    if (o.mixed) recip_of(o.mixed, &o.mul, &o.shift);
    return true;
}
inline uint32_t stream_groups(int tiles) { return (uint32_t)(tiles + 7) / 8u + 1u; }      // of an operand's first pass: its tiles, and the one that collects

// Groups of eight workgroups spread evenly among others.
struct Spread {
    uint32_t n, mul, shift;       // that many among a number of groups; reciprocal of that number
};
__device__ __forceinline__ uint32_t spread_before(const Spread& s, uint32_t group) { return recip_div(group * s.n, s.mul, s.shift); }
inline bool spread_fits(uint64_t n, uint64_t all) { return n <= all && all < 0x7FFFFFFFull && (all + 1) * n < 0x7FFFFFFFull; }      // (see recip_div)
inline bool make_spread(Spread& s, uint32_t n, uint32_t all) {
    s.n = n;
    recip_of(all ? all : 1u, &s.mul, &s.shift);
    return spread_fits(n, all);
}

// `Tile`: count(tile, lane of the workgroup, amax, flushes) adds a lane's share of a tile to its figures, `amax` a pattern.
__device__ __forceinline__ uint32_t stream_tile_word(uint32_t amax, uint32_t flushes) { return kThere | (flushes << kFlushShift) | amax; }
template <class Tile>
__device__ __forceinline__ void stream_first(uint32_t* words, int tile, uint32_t* sh8, Tile count) {
    uint32_t amax = 0u, flushes = 0u;
    count(tile, (int)threadIdx.x, amax, flushes);
    amax = wave_allmax_u32(amax);
    flushes = wave_allsum_u32(flushes);
    if ((threadIdx.x & 63) == 0) { sh8[threadIdx.x >> 6] = amax; sh8[4 + (threadIdx.x >> 6)] = flushes; }
    __syncthreads();
    if (threadIdx.x == 0)
        agent_store(words + kStreamTiles + tile, stream_tile_word(max(max(sh8[0], sh8[1]), max(sh8[2], sh8[3])), (sh8[4] + sh8[5]) + (sh8[6] + sh8[7])));
}
__device__ __forceinline__ uint32_t stream_figures(uint32_t amax, uint32_t flushes, uint32_t flush_need) {
    return kThere | (flush_need != 0u && flushes >= flush_need ? kToldProven : 0u) | amax;
}
// Where wave w of a unit's workgroup begins its scan: the waves of neighbouring units far from each other.
__device__ __forceinline__ uint32_t stream_scan_from(uint32_t unit, int tiles) {
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(unit * 4u + (threadIdx.x >> 6)));
    return __umulhi(wave * 0x9E3779B1u, (uint32_t)tiles);
}
// The operand's figures by a wave of its own, beginning at tile `from` (an operand has less than 2^32 elements).  A tile whose word is there is
// not read; one that is not is counted and its word left, the same that its workgroup leaves, and the figures are told.  So however many
// waves are here, together they read what of the operand has not been read yet, and little of it twice; each of them, its words.
// us per call as it is / where no wave waits at all: per-tensor 8192 x 4096 42.5 / 260, 8192 x 14336 with padded rows 110 / 335, two of these
// dense 189 / 502, 128 x 128 blocks of 8192 x 8192 69 / 327, twelve of 8192 x 4096 by rows 286 / 1116.  (Each wave going through all tiles, as
// it was, would read 64 MB for each of 8192 waves in the first.)
template <class Tile>
__device__ __forceinline__ uint32_t stream_scan(uint32_t* words, int tiles, uint32_t from, uint32_t flush_need, Tile count) {
    const int lane = (int)(threadIdx.x & 63u), chunks = (tiles + 63) >> 6, turn = (int)(from & 63u);
    uint32_t amax = 0u, flushes = 0u;
    int c = (int)(from >> 6);                              // chunks of 64 words, one per lane
#pragma clang loop unroll(disable)
    for (int k = 0; k < chunks; ++k) {
        const int i = c * 64 + lane;
        uint32_t v = i < tiles ? 0u : kThere;
#pragma clang loop unroll(disable)
        for (;;) {                                         // a turn adds a word at least
            if (!(v & kThere)) v = agent_load(words + kStreamTiles + i);
            const unsigned long long missing = __ballot(!(v & kThere));
            if (missing == 0ull) break;
            const unsigned long long turned = turn ? (missing >> turn) | (missing << (64 - turn)) : missing;
            const int at = (__builtin_ctzll(turned) + turn) & 63;
            uint32_t a = 0u, f = 0u;
#pragma clang loop unroll(disable)
            for (int part = 0; part < 4; ++part) count(c * 64 + at, part * 64 + lane, a, f);
            const uint32_t word = stream_tile_word(wave_allmax_u32(a), wave_allsum_u32(f));
            if (lane == at) { v = word; agent_store(words + kStreamTiles + i, word); }
        }
        amax = max(amax, v & kAmaxBits);                   // (lanes beyond the last tile: zeros)
        flushes += (v & ~kThere) >> kFlushShift;
        if (++c == chunks) c = 0;
    }
    const uint32_t figures = stream_figures(wave_allmax_u32(amax), wave_allsum_u32(flushes), flush_need);
    if (lane < kToldCopies) agent_store(words + lane * kToldLine, figures);
    return figures;
}
// By the workgroup that collects: from the tiles' words, which it tells; the same value in all lanes.
template <class Tile>
__device__ __forceinline__ uint32_t stream_collect(uint32_t* words, int tiles, uint32_t flush_need, int polls, uint32_t* sh8, Tile count) {
    const int tid = threadIdx.x;
    uint32_t amax = 0u, flushes = 0u;
    bool all = true;
    for (int i0 = tid; i0 < tiles; i0 += 8 * 256) {
        uint32_t v[8];
        for (;;) {
            uint32_t there = kThere;
#pragma unroll
            for (int u = 0; u < 8; ++u) { v[u] = agent_load(words + kStreamTiles + (i0 + u * 256 < tiles ? i0 + u * 256 : i0)); there &= v[u]; }
            all = there != 0u;
            if (all || polls-- <= 0) break;
            __builtin_amdgcn_s_sleep(8);
        }
        if (!all) break;
#pragma unroll
        for (int u = 0; u < 8; ++u) { amax = max(amax, v[u] & kAmaxBits); flushes += i0 + u * 256 < tiles ? (v[u] & ~kThere) >> kFlushShift : 0u; }
    }
    amax = wave_allmax_u32(amax);
    flushes = wave_allsum_u32(flushes);
    if ((tid & 63) == 0) { sh8[tid >> 6] = amax; sh8[4 + (tid >> 6)] = flushes; }
    const bool every = __syncthreads_and(all ? 1 : 0) != 0;
    if (!every) return stream_scan(words, tiles, stream_scan_from(0u, tiles), flush_need, count);
    const uint32_t figures = stream_figures(max(max(sh8[0], sh8[1]), max(sh8[2], sh8[3])), (sh8[4] + sh8[5]) + (sh8[6] + sh8[7]), flush_need);
    if (tid < kToldCopies) agent_store(words + tid * kToldLine, figures);
    return figures;
}
// What a wave is told, `look` being what it has seen first; 0 if that does not come in time.
__device__ __forceinline__ uint32_t stream_told(const uint32_t* copy, uint32_t look, int polls) {
    uint32_t told = (uint32_t)__builtin_amdgcn_readfirstlane((int)look);
    for (int poll = 0; poll < polls && !(told & kThere); ++poll) {
        __builtin_amdgcn_s_sleep(8);
        told = (uint32_t)__builtin_amdgcn_readfirstlane((int)agent_load(copy));
    }
    return told & kThere ? told : 0u;
}
__device__ __forceinline__ const uint32_t* stream_copy(const uint32_t* words, int64_t unit) { return words + (unit & (kToldCopies - 1)) * kToldLine; }
// The words are cleared by a launch before: 4 KB per workgroup.
__device__ __forceinline__ void stream_clear(uint32_t* words, int tiles, int b) {
    const int i = (b * 256 + (int)threadIdx.x) * 4;
    if (i < kStreamTiles + tiles) *reinterpret_cast<u32x4*>(words + i) = u32x4{0u, 0u, 0u, 0u};
}
inline unsigned stream_clear_wgs(int tiles) { return (unsigned)((kStreamTiles + tiles + 1023) / 1024); }

}  // namespace mor
