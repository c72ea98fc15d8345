// sc_kernels.hip -- gfx950 kernels of the strip unpacking + three-threshold clustering path.
//
// Paper §2 (Parallelization): FEDs of 96 channels x 256 strips; ZS data stored per FED like CSR
// (channel = row, strip = column); unpacking concurrently per channel; clustering by seed seeking
// over strips, then cluster forming over seeds. §3 (Optimization): several events in flight.
//
// MI355X design (not the paper's CUDA design):
//  * a workgroup of W wavefronts owns one (event, FED) tile at a time; a persistent grid pulls
//    tiles from an atomic queue, FED-major (the events of one FED back to back, so its
//    calibration is reused from cache) or event-major, or from eight FED-major queues with the
//    FEDs dealt round-robin, one queue per XCD (workgroup i runs on XCD i mod 8): the events of
//    a FED then run on one XCD and its calibration is fetched into one L2, not eight;
//  * the FED's bytes and gains are staged into LDS with all 16-byte loads in flight at once; wave
//    0 walks the 96 length fields in LDS (the channel map the paper builds on the CPU); then each
//    wave takes a group of 96/W channels on its own: one lane per channel validates the records
//    and marks where each begins in the wave's digi list in LDS, from which forming takes the digis;
//  * cluster forming runs digi-parallel, in windows of 256 digis (four per lane), with the next
//    window's calibration gathers in flight: the active/seed tests use one FP32 effective noise
//    per strip (+inf for unusable strips, which never passes ADC > T*noise); a run is a chain of
//    active digis on adjacent strips, found with wave masks, and its sums (noise squares, charge,
//    seeds) go along the four digis of a lane and from lane to lane, in the definition's order;
//  * the waves exchange their groups' counts in LDS; the tile publishes the FED's counts and looks
//    back over the earlier FEDs of its event, 64 per load (decoupled look-back), for its output
//    offsets; forming leaves the list of cluster members, from which records are written by the
//    lane of each cluster's last strip and member ADCs (gain-corrected here) four per lane, again
//    in windows of 256; the writes of a tile come after the first half of the next.
// No MFMA: nothing here is a dense contraction.

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "sc_internal.h"

// The allocation-free batch call's scratch (layout in sc_internal.h). Host code must not use this
// name as an address: it reaches the array through static_scratch_address().
static __device__ __align__(256) unsigned char scratch[sc::kStaticScratchBytes];

namespace sc {

hipError_t static_scratch_address(void** ptr) {
    return hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch));
}

namespace {

constexpr uint32_t kSpinLimit = 1u << 22;   // look-back wait bound (seconds of sleeping)
constexpr uint32_t kWalkPolls = 6;          // look-back polls that fit beside a walk
constexpr uint32_t kXcdShift = 3;           // 8 XCDs (queues of tile order 2)
constexpr uint32_t kXcds = 1u << kXcdShift;
constexpr int kNch = kChannelsPerFed;
constexpr int kStripsPerFed = kChannelsPerFed * kStripsPerChannel;

// ---- global-address-space views (plain global loads/stores, no flat addressing) ------------
#ifndef SC_GLOBAL_AS
#define SC_GLOBAL_AS __attribute__((address_space(1)))
#endif
template <class T> using gconst = SC_GLOBAL_AS const T;
template <class T> using gmut = SC_GLOBAL_AS T;
template <class T> __device__ __forceinline__ gconst<T>* gc(const T* p) { return (gconst<T>*)p; }
template <class T> __device__ __forceinline__ gmut<T>* gm(T* p) { return (gmut<T>*)p; }

// The element `bytes` past a uniform base: a scalar base and one 32-bit offset, no 64-bit addition
// per lane. (An event has at most 20000 x 96 channels of 128 clusters: 16 bytes each stay below 2^32.)
template <class T> __device__ __forceinline__ gmut<T>* at_offset(gmut<T>* base, uint32_t bytes) {
    return reinterpret_cast<gmut<T>*>(reinterpret_cast<gmut<uint8_t>*>(base) + bytes);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // 16-byte global accesses
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u32x2 u32x2_by2 __attribute__((aligned(2)));          // at any even address

__device__ __forceinline__ uint32_t lane() { return __lane_id(); }
// x + the set bits of the wave mask m below this lane (v_mbcnt)
__device__ __forceinline__ uint32_t count_below(uint64_t m, uint32_t x) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, x));
}
__device__ __forceinline__ uint32_t popc(uint64_t m) { return (uint32_t)__popcll(m); }
__device__ __forceinline__ uint32_t uni(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ uint64_t uni64(uint64_t v) {
    return (uint64_t)uni((uint32_t)v) | ((uint64_t)uni((uint32_t)(v >> 32)) << 32);
}
template <class T> __device__ __forceinline__ T* uniptr(T* p) {
    return reinterpret_cast<T*>(uni64(reinterpret_cast<uintptr_t>(p)));
}
// value of lane 63, as a uniform value
__device__ __forceinline__ uint32_t last_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}
// Lane i receives lane i-1's value (lane 0 receives 0): DPP wave_shr:1.
__device__ __forceinline__ uint32_t from_prev_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, false);
}
// Lane i receives lane i+1's value (lane 63 receives 0): DPP wave_shl:1.
__device__ __forceinline__ uint32_t from_next_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, false);
}

template <int Ctrl, int RowMask>
__device__ __forceinline__ uint32_t dpp_in(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, Ctrl, RowMask, 0xf, true);
}
// Inclusive sum over the wavefront in six DPP steps: row_shr 1, 2, 4, 8 inside rows of 16 lanes,
// then row_bcast:15 into rows 1 and 3 and row_bcast:31 into rows 2 and 3.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
    x += dpp_in<0x111, 0xf>(x);
    x += dpp_in<0x112, 0xf>(x);
    x += dpp_in<0x114, 0xf>(x);
    x += dpp_in<0x118, 0xf>(x);
    x += dpp_in<0x142, 0xa>(x);
    x += dpp_in<0x143, 0xc>(x);
    return x;
}

// Inclusive maximum over the wavefront, in the same six DPP steps (out-of-row sources read 0).
__device__ __forceinline__ uint32_t wave_incl_max(uint32_t x) {
    x = __builtin_elementwise_max(x, dpp_in<0x111, 0xf>(x));
    x = __builtin_elementwise_max(x, dpp_in<0x112, 0xf>(x));
    x = __builtin_elementwise_max(x, dpp_in<0x114, 0xf>(x));
    x = __builtin_elementwise_max(x, dpp_in<0x118, 0xf>(x));
    x = __builtin_elementwise_max(x, dpp_in<0x142, 0xa>(x));
    x = __builtin_elementwise_max(x, dpp_in<0x143, 0xc>(x));
    return x;
}

__device__ __forceinline__ uint32_t wave_excl_scan(uint32_t v, uint32_t& total) {
    const uint32_t x = wave_incl_scan(v);
    total = last_lane(x);
    return x - v;
}

__device__ __forceinline__ uint32_t seg16_excl_scan(uint32_t v, uint32_t& total) {
    uint32_t x = v;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
        uint32_t y = __shfl_up(x, d, 16);
        if ((int)(lane() & 15) >= d) x += y;
    }
    total = __shfl(x, 15, 16);
    return x - v;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return last_lane(wave_incl_scan(v)); }

// Control-flow rule of these kernels: no branch on a lane-dependent, loop-invariant condition
// (lane() == 0 and the like) around the persistent tile loop or the chunk loops. The middle end
// may thread two such branches across a loop back edge; the loop then splits into an inner loop
// for some lanes of the wavefront and an outer one for the others, which a SIMD machine runs as
// a deadlock. Work done "by one lane" is instead done by every lane with identical values, lane
// tests only select values, and every tile ends at a barrier. Branches on the wave index are
// uniform per wavefront; workgroup barriers sit only where every wave passes (tile level).

// ---- look-back words: flag(2) | n_cl(31) | n_adc(31) -------------------------------------
constexpr uint64_t kFlagAgg = 1, kFlagIncl = 2;
__device__ __forceinline__ unsigned long long pack_state(uint64_t flag, uint32_t ncl,
                                                         uint32_t nadc) {
    return (flag << 62) | ((uint64_t)(ncl & 0x7fffffffu) << 31) | (uint64_t)(nadc & 0x7fffffffu);
}

// The digi list of a wave holds, while a channel group is built and formed,
//  * markers, in the slot of each ZS record's first digi: bit 31, and
//      (source << 17 | position << 2) - slot * kSlotStep   (+ kMaybeBit),
//    source = the stage offset of the digi's ADC byte, position = channel-in-FED * 256 + strip.
//    Adding slot' * kSlotStep gives source and position of any later digi of the record, at slot';
//  * digi words: position << 10 | ADC.
// Once formed, it holds the words of the members of accepted clusters alone, close together from its
// start, with kContBit on each but the first of a cluster.
constexpr uint32_t kSlotStep = 1u << 17 | 4u, kMarker = 1u << 31, kMaybeBit = 1u;
constexpr uint32_t kContBit = 1u << 29;
constexpr uint32_t kNoStrip = 0xffffffffu;
constexpr uint32_t kNoiseMask = 0x1fffcu;   // position << 2: byte offset in the FED's noise table
__device__ __forceinline__ uint32_t d_adc(uint32_t d) { return d & 255u; }
__device__ __forceinline__ uint32_t d_strip(uint32_t d) { return (d >> 10) & 255u; }
__device__ __forceinline__ uint32_t d_ch(uint32_t d) { return (d >> 18) & 127u; }
__device__ __forceinline__ uint32_t d_pos(uint32_t d) { return (d >> 10) & 0x7fffu; }
// x * y + z for x, y < 2^24 (a full-rate instruction; v_mul_lo_u32 runs at a quarter of it)
__device__ __forceinline__ uint32_t mad24(uint32_t x, uint32_t y, uint32_t z) {
    return __umul24(x, y) + z;
}
// a lane's bit of a wave mask, as a select condition
__device__ __forceinline__ bool in_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Module rows (tiles instantiated with kMod): bit c of the FED's join words is set when channel c
// reads the same module as channel c - 1, whose strips then continue into it (strip 255 of c - 1
// is followed by strip 0 of c; positions ch * 256 + strip stay consecutive across the edge).
// A row has at most 3 channels (768 strips) and never crosses a multiple of 24 channels, so the
// wave groups and the chunks of a group hold whole rows.
struct Joins {
    uint32_t w0, w1, w2;
};
__device__ __forceinline__ bool joined(Joins J, uint32_t ch) {
    const uint32_t w = ch < 32u ? J.w0 : ch < 64u ? J.w1 : J.w2;
    return ((w >> (ch & 31u)) & 1u) != 0u;
}
// Raw ADC sum | seed count << kQShift in one word: a channel run's sum fits 16 bits (256 x 255),
// a module row's needs 18 (768 x 255).
template <bool kMod> constexpr uint32_t kQShift = kMod ? 18u : 16u;

// LDS stage sizes: the small one holds a FED of full-detector events at 5 % occupancy, the
// large one (fewer resident tiles) a FED of the 6 %, long-cluster stress events.
constexpr int kStageSmall = 6656, kStageLarge = 10240;

// A wave's list is read four words at a time from any slot below its end, and cleared in 16-byte
// pieces: four words of pad, of which three are read.
constexpr int kListPad = 4;

template <int W, int DW, int S = kStageSmall>
struct TileSmem {
    static constexpr int kStageBytes = S;
    static constexpr int kStageData = kStageBytes - 16;   // FED bytes that fit (alignment slack)
    static constexpr int kList = DW + kListPad;
    alignas(16) float gain[4 * kNch];                    // the FED's APV gains and reciprocals, in pairs
    alignas(16) uint8_t stage[kStageBytes + 4];          // the FED's bytes (+ readable pad)
    alignas(16) uint32_t digi[W * kList];                // wave w: [w * kList, w * kList + DW)
    uint32_t ch_pos[kNch + 2];    // payload positions; [96]: past the last record, + 2; [97]: unused
    uint16_t ch_base[kNch + W];   // channel c of wave w at index c + w: digi offset in the group,
                                  // and kChBad if its record is malformed
    // chunks of a group: two in a row hold more than DW digis, so there are few
    static constexpr int kGroupChans = kNch / W;
    static constexpr int kMaxChunks = 2 * kGroupChans * kStripsPerChannel / DW + 1 < kGroupChans
                                          ? 2 * kGroupChans * kStripsPerChannel / DW + 1
                                          : kGroupChans;
    uint8_t chunk_first[W][kMaxChunks + 1];
    uint32_t walk[2];             // bad_from, trailing
    uint32_t next[5];             // the next tile: event (kNoTile: none), FED, bytes, address
    uint32_t grp_cnt[W + 1][3];   // per group: clusters, member ADCs, chunks; [W]: the FED's
                                  // offsets, look-back failure
};
constexpr uint32_t kNoTile = 0xffffffffu;
constexpr uint32_t kChBad = 0x8000u;

// Two-wave tiles of 2880 digis fit eight to a CU (160 KiB of LDS).
static_assert(sizeof(TileSmem<2, 1440>) <= 160 * 1024 / 8, "eight two-wave tiles per CU");
static_assert(sizeof(TileSmem<2, 1440, kStageLarge>) <= 160 * 1024 / 6, "six with the large stage");

// Workgroup barrier (every wave of the tile passes it); a no-op for single-wave tiles.
__device__ __forceinline__ void tile_sync() { __syncthreads(); }
// Orders this wavefront's LDS accesses (lanes of one wave see each other's earlier stores).
__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

// Index of the calling wave in the tile, as a uniform (scalar) value.
template <int W>
__device__ __forceinline__ uint32_t wave_index() {
    if constexpr (W == 1) return 0u;
    else return uni(threadIdx.x >> 6);
}

// The APV gains of a wave's channels (pairs of gain and reciprocal), as 16-byte vectors.
template <int W>
struct GainVecs {
    static constexpr uint32_t kCount = kNch / W;   // 4 floats per channel
    static constexpr int kPerLane = (kCount + kWave - 1) / kWave;
    u32x4 v[kPerLane];
};
// (lanes past the last vector repeat it)
template <int W>
__device__ __forceinline__ uint32_t gain_index(int i) {
    const uint32_t k = (uint32_t)i * kWave + lane();
    return k < GainVecs<W>::kCount ? k : GainVecs<W>::kCount - 1u;
}
template <int W>
__device__ __forceinline__ void load_gains(GainVecs<W>& g, const float* gains, uint32_t fed, uint32_t w) {
    gconst<u32x4>* src = gc(reinterpret_cast<const u32x4*>(gains)) + fed * kNch + w * GainVecs<W>::kCount;
#pragma unroll
    for (int i = 0; i < GainVecs<W>::kPerLane; ++i) g.v[i] = src[gain_index<W>(i)];
}
template <int W, int DW, int S>
__device__ __forceinline__ void store_gains(TileSmem<W, DW, S>& sm, const GainVecs<W>& g, uint32_t w) {
    u32x4* dst = reinterpret_cast<u32x4*>(sm.gain) + w * GainVecs<W>::kCount;
#pragma unroll
    for (int i = 0; i < GainVecs<W>::kPerLane; ++i) dst[gain_index<W>(i)] = g.v[i];
}

// ---- staging -----------------------------------------------------------------------------
// The 16-byte aligned pieces that cover bytes [src, src + n), n <= kStageBytes - 15, held by NT
// threads (t: the thread's index), all loaded before the first is put into the stage, where src[i]
// lands at stage[delta + i]. Every piece holds at least one byte of the range, so it lies inside
// the 4 KiB page of a byte of the buffer.
template <int S, int NT>
struct Pieces {
    static constexpr int K = (S + 16 * NT - 1) / (16 * NT);
    u32x4 r[K];
    static __device__ __forceinline__ uint32_t delta(const uint8_t* src) {
        return (uint32_t)(reinterpret_cast<uintptr_t>(src) & 15u);
    }
    static __device__ __forceinline__ uint32_t count(const uint8_t* src, uint32_t n) {
        return n ? (delta(src) + n + 15u) >> 4 : 0u;
    }
    __device__ __forceinline__ void load(const uint8_t* src, uint32_t n, uint32_t t) {
        const uint32_t pieces = count(src, n);
        if (!pieces) return;
        // every thread loads K pieces (indices past the end repeat the last piece)
        const uint32_t last = pieces - 1u;
        gconst<u32x4>* s4 = gc(reinterpret_cast<const u32x4*>(src - delta(src)));
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t c = t + (uint32_t)(k * NT);
            r[k] = s4[c < last ? c : last];
        }
    }
    __device__ __forceinline__ void store(uint8_t* stage, const uint8_t* src, uint32_t n,
                                          uint32_t t) const {
        const uint32_t pieces = count(src, n);
        u32x4* d4 = reinterpret_cast<u32x4*>(stage);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint32_t c = t + (uint32_t)(k * NT);
            if (c < pieces) d4[c] = r[k];
        }
    }
};

// ---- channel map: the 96 length fields (uniform walk by wave 0) ----------------------------
struct WalkResult {
    uint32_t bad_from;   // first channel failing the record-in-FED rule (96: none)
    uint32_t trailing;   // 1 if bytes follow the 96th record
    uint32_t fits;       // 1 if the whole FED is in the stage, and the payload positions count
                         // from the stage's start (else from the FED's)
};

// Walks the length fields of a FED of L bytes that lies in the stage from delta on; by one wave.
template <int W, int DW, int S>
__device__ __forceinline__ void walk_staged(TileSmem<W, DW, S>& sm, uint32_t delta, uint32_t L) {
    // Lane k (mod 64) keeps channel k's payload position in the stage. Branch-free steps
    // whose serial chain is only clamp, read, two adds (vector instructions, uniform
    // values): 96 LDS round trips, which bound a tile that is alone on its CU. Record k
    // ends where record k + 1's length field starts, so the fit test comes from the
    // positions afterwards: a record fits the FED when its end is <= the FED's, and since
    // ends only grow, the records that fit come first (past the first one that does not,
    // the reads stay inside the stage and are unused). Ends stay below 2^23 (96 x (2 +
    // 65535)): no sum wraps.
    constexpr uint32_t omax = TileSmem<W, DW, S>::kStageBytes + 2;   // two readable bytes before it
    const uint32_t fed_end = delta + L;
    uint32_t pos = delta + 2u;   // past the length field of record k
    uint32_t vpos0 = 0, vpos1 = 0;
    auto step = [&](uint32_t k, uint32_t& vpos) {
        const uint32_t o = pos < omax ? pos : omax;
        // the chain stays in vector registers (the empty asm keeps the bytes there): the
        // CU's one scalar unit, shared by its four SIMDs, is busy with the other waves'
        // scalar work, and a scalar chain would wait for it at every step
        uint32_t lo = sm.stage[o - 2u], hi = sm.stage[o - 1u];
        // (what does not wait for the bytes goes before them: 20 events of 440 FEDs 97 -> 94.5 us, 64
        // 283 -> 278. One 16-bit read at an odd address instead of two of a byte: 118 and 326.)
        vpos = __builtin_amdgcn_inverse_ballot_w64(1ull << (k & 63u)) ? pos : vpos;
        uint32_t next = pos + 2u;
        asm volatile("" : "+v"(lo), "+v"(hi), "+v"(next), "+v"(vpos));
        pos = (hi << 8) + lo + next;
    };
#pragma unroll 8
    for (uint32_t k = 0; k < 64u; ++k) step(k, vpos0);
#pragma unroll 8
    for (uint32_t k = 64; k < (uint32_t)kNch; ++k) step(k, vpos1);
    constexpr uint32_t kLast = (uint32_t)kNch - 65u;   // lane of channel 95 in vpos1
    const uint32_t l = lane();
    // lane 32: where record 95 ends, as a payload position
    vpos1 = l == kLast + 1u ? pos : vpos1;
    // (the cross-lane reads are taken by every lane first: inside a conditional
    // expression they would run under a partial exec mask, and a DPP read from a
    // disabled lane returns the fallback value)
    const uint32_t next1 = (uint32_t)__builtin_amdgcn_readlane((int)vpos1, 0);
    const uint32_t nx0 = from_next_lane(vpos0), nx1 = from_next_lane(vpos1);
    const uint32_t end0 = (l == 63u ? next1 : nx0) - 2u, end1 = nx1 - 2u;
    const uint32_t good = popc(__ballot(end0 <= fed_end)) +
                          popc(__ballot(l <= kLast && end1 <= fed_end));
    sm.ch_pos[l] = vpos0;
    // (the lanes past channel 95's end write the unused entry)
    sm.ch_pos[l <= kLast + 1u ? 64u + l : (uint32_t)kNch + 1u] = vpos1;
    sm.walk[0] = good;
    sm.walk[1] = (good == (uint32_t)kNch && pos - 2u < fed_end) ? 1u : 0u;
}

// The same for a FED larger than the stage: windows of it are staged in turn; the records are then
// read from global memory.
template <int W, int DW, int S>
__device__ __forceinline__ void walk_windows(TileSmem<W, DW, S>& sm, const uint8_t* g, uint32_t L) {
    constexpr uint32_t cap = TileSmem<W, DW, S>::kStageData;
    uint32_t pos = 0, bad_from = kNch, win = 0, win_n = 0, delta = 0;
    for (uint32_t k = 0; k < (uint32_t)kNch; ++k) {
        if (pos + 2 > L) { bad_from = k; break; }
        if (pos + 2 > win + win_n) {
            wave_sync();
            win = pos;
            win_n = (L - win) < cap ? (L - win) : cap;
            Pieces<TileSmem<W, DW, S>::kStageBytes, kWave> p;
            p.load(g + win, win_n, lane());
            p.store(sm.stage, g + win, win_n, lane());
            delta = p.delta(g + win);
            wave_sync();
        }
        const uint32_t o = pos - win + delta;
        const uint32_t P = uni((uint32_t)sm.stage[o] | ((uint32_t)sm.stage[o + 1] << 8));
        if (pos + 2 + P > L) { bad_from = k; break; }
        sm.ch_pos[k] = pos + 2;   // the same values from every lane
        pos += 2 + P;
    }
    sm.ch_pos[bad_from] = pos + 2;   // where record bad_from - 1 ends
    sm.walk[0] = bad_from;
    sm.walk[1] = (bad_from == (uint32_t)kNch && pos < L) ? 1u : 0u;
}

// Whether a FED of L bytes is staged whole.
template <int W, int DW, int S>
__device__ __forceinline__ bool fits_stage(const TileSmem<W, DW, S>&, uint32_t L) {
    return L <= (uint32_t)TileSmem<W, DW, S>::kStageData;
}

template <int W, int DW, int S>
__device__ __forceinline__ void walk_fed(TileSmem<W, DW, S>& sm, const uint8_t* g, uint32_t L) {
    __builtin_amdgcn_s_setprio(3);   // the tile's other waves wait for it
    if (fits_stage(sm, L)) walk_staged(sm, Pieces<S, kWave * W>::delta(g), L);
    else walk_windows(sm, g, L);
    __builtin_amdgcn_s_setprio(2);
}

template <int W, int DW, int S>
__device__ __forceinline__ WalkResult walk_result(const TileSmem<W, DW, S>& sm, uint32_t L) {
    return WalkResult{uni(sm.walk[0]), uni(sm.walk[1]), fits_stage(sm, L) ? 1u : 0u};
}

// Payload bytes of channel ch (below the walk's bad_from): its record ends where the next begins.
template <int W, int DW, int S>
__device__ __forceinline__ uint32_t payload_len(const TileSmem<W, DW, S>& sm, uint32_t ch) {
    return sm.ch_pos[ch + 1] - 2u - sm.ch_pos[ch];
}

// ---- record validation, one lane per channel ----------------------------------------------
// Returns the channel's digi count, or kChBad if it is malformed; near: the smallest distance of a
// record's first strip from the end of the record before it (0: they are adjacent; `on`: the first
// record's is taken from strip 0). Inside the loop a record is only tested for order and for holding
// a digi: then the strips only grow, and that the last record ends at the channel's end or before,
// and at the payload's end, is seen after it. A valid channel has at most 256 records of 3 bytes, so
// no longer payload is walked. The loop's chain is one LDS round trip, an addition and the compare
// with the payload's end; with a branch for each rule an iteration took 440 cycles on an idle CU.
template <class P, int W, int DW, int S>
__device__ __forceinline__ uint32_t check_channel(TileSmem<W, DW, S>& sm, P src, uint32_t ch,
                                                  const WalkResult& w, bool on, uint32_t& near) {
    constexpr bool kStaged = std::is_same_v<P, const uint8_t*>;
    if (ch >= w.bad_from) return kChBad;
    uint32_t a = sm.ch_pos[ch];
    const uint32_t n = payload_len(sm, ch), end = a + n;
    if (n > 3u * kStripsPerChannel) return kChBad;
    uint32_t nd = 0u, free = 0u, gap = kNoStrip;
    int32_t bad = 0;
    // the strip that the next record may start on; the first one's distance from it is not 0
    // unless it may go on from the channel before
    uint32_t next_free = on ? 0u : kNoStrip;
    while (a < end) {
        // (the second byte of a dangling header is the next length field's, or the stage's pad; in
        // global memory it may lie past the buffer, and any byte in its place ends the same)
        const uint32_t first = src[a], cnt = src[kStaged || a + 1u < end ? a + 1u : a];
        const uint32_t d = first - next_free;
        bad |= (int32_t)(d | (cnt - 1u));
        gap = __builtin_elementwise_min(gap, d);
        next_free = free = first + cnt;
        nd += cnt;
        a += 2u + cnt;
    }
    near = gap;
    const bool wrong = (bad < 0) | (free > (uint32_t)kStripsPerChannel) | (a != end);
    return wrong ? kChBad : nd;
}

// Digi offset of entry i of the channel table (channel c of wave w: c + w) in its group.
template <int W, int DW, int S>
__device__ __forceinline__ uint32_t digi_base(const TileSmem<W, DW, S>& sm, uint32_t i) {
    return sm.ch_base[i] & ~kChBad;
}

// The channel group [c_lo, c_hi) of wave w: digi counts -> offsets in the group (ch_base) and
// its split into chunks of at most DW digis; returns the number of chunks and whether any channel is
// malformed, and any record may go on from the one before it: its first strip follows that one's last
// (runs of more than 255 strips are written so) or, in a module row, is strip 0 of a joined
// channel. Wave-local.
template <bool kMod, int W, int DW, int S, class CountFn>
__device__ uint32_t plan_chunks(TileSmem<W, DW, S>& sm, uint32_t w, uint32_t c_lo, uint32_t c_hi,
                                Joins J, CountFn count, bool& any_bad, bool& any_on) {
    uint32_t carry = 0;
    any_bad = any_on = false;
    for (uint32_t base = c_lo; base < c_hi; base += kWave) {
        const uint32_t ch = base + lane();
        uint32_t near = kNoStrip;
        const bool on = kMod && joined(J, ch);
        const uint32_t nd = ch < c_hi ? count(ch, on, near) : 0u;   // kChBad: malformed, no digis
        uint32_t tot;
        const uint32_t ex = wave_excl_scan(nd & ~kChBad, tot);
        if (ch < c_hi) sm.ch_base[ch + w] = (uint16_t)((carry + ex) | (nd & kChBad));
        carry += tot;
        any_bad |= __ballot((nd & kChBad) != 0u) != 0ull;
        any_on |= __ballot(near == 0u) != 0ull;
    }
    const uint32_t total = carry;
    sm.ch_base[c_hi + w] = (uint16_t)carry;   // uniform stores from every lane
    uint8_t* cf = sm.chunk_first[w];
    uint32_t n_chunks = 1;
    wave_sync();
    if (total <= (uint32_t)DW) {
        cf[0] = (uint8_t)c_lo;
        cf[1] = (uint8_t)c_hi;
    } else {
        // every lane walks the same greedy split (uniform values, same stores)
        uint32_t c = c_lo, n = 0;
        cf[0] = (uint8_t)c_lo;
        while (c < c_hi) {
            const uint32_t start = uni(digi_base(sm, c + w));
            if constexpr (kMod) {
                // whole rows only: a row holds <= 768 <= DW digis (the host keeps DW >= 768)
                uint32_t c1 = c + 1;
                while (c1 < c_hi && joined(J, c1)) ++c1;
                while (c1 < c_hi) {
                    uint32_t c2 = c1 + 1;
                    while (c2 < c_hi && joined(J, c2)) ++c2;
                    if (uni(digi_base(sm, c2 + w)) - start > (uint32_t)DW) break;
                    c1 = c2;
                }
                cf[++n] = (uint8_t)c1;
                c = c1;
            } else {
                uint32_t c1 = c + 1;   // one channel holds <= 256 <= DW digis
                while (c1 < c_hi && uni(digi_base(sm, c1 + 1 + w)) - start <= (uint32_t)DW) ++c1;
                cf[++n] = (uint8_t)c1;
                c = c1;
            }
        }
        n_chunks = n;
    }
    wave_sync();
    return n_chunks;
}

// The records of channels [c0, c1) of a staged FED, as markers in the digi list dl (one lane per
// channel). any_on (uniform): some record may go on from the one before it, and such records get
// kMaybeBit.
// Records take their slots in the order of their bytes, and from one record to the next the source
// grows by the first one's digis plus a 2-byte header, the slot by the digis alone: the source
// field, and with it the marker, grows, and the last marker at or before a slot is the largest.
template <bool kMod, int W, int DW, int S>
__device__ __forceinline__ void build_markers(TileSmem<W, DW, S>& sm, uint32_t w, uint32_t* dl,
                                              Joins J, bool any_on, uint32_t c0, uint32_t c1) {
    static_assert(TileSmem<W, DW, S>::kStageBytes + 16 < (1 << 14), "marker sources are 14 bits");
    static_assert(DW * 4 < (1 << 18), "position - slot must not borrow past one source step");
    const uint32_t b0 = digi_base(sm, c0 + w);
    const uint32_t nd = digi_base(sm, c1 + w) - b0;
    static_assert(DW % 4 == 0 && TileSmem<W, DW, S>::kList % 4 == 0, "lists of whole 16-byte pieces");
    // (what the list held before may look like markers)
    for (uint32_t o = 4u * lane(); o < nd; o += 4u * kWave)
        *reinterpret_cast<u32x4*>(dl + o) = u32x4{0u, 0u, 0u, 0u};
    __builtin_amdgcn_s_setprio(2);   // a serial pass that the digi pass waits for
    for (uint32_t ch = c0 + lane(); ch < c1; ch += kWave) {
        const uint32_t bw = sm.ch_base[ch + w];
        // (a channel past the walk's last good one has no position)
        uint32_t a = (bw & kChBad) ? 0u : sm.ch_pos[ch];
        const uint32_t end = (bw & kChBad) ? 0u : a + payload_len(sm, ch);
        uint32_t o = bw - b0;
        // source - slot grows by the two header bytes from record to record
        uint32_t m = kMarker + ((a + 2u - o) << 17) + (ch << 10);
        // each record's header is read while the one before is put down (the last read is of the
        // bytes after the channel, unused)
        uint32_t first = sm.stage[a], cnt = sm.stage[a + 1u];
        auto records = [&](auto with_on, uint32_t next) {
            while (a < end) {
                a += 2u + cnt;
                const uint32_t first2 = sm.stage[a], cnt2 = sm.stage[a + 1u];
                uint32_t marker = m + ((first - o) << 2);
                if constexpr (decltype(with_on)::value) {
                    marker += first == next ? kMaybeBit : 0u;
                    next = first + cnt;
                }
                dl[o] = marker;
                m += 2u << 17;
                o += cnt;
                first = first2;
                cnt = cnt2;
            }
        };
        if (any_on) records(std::true_type{}, kMod && joined(J, ch) ? 0u : kNoStrip);
        else        records(std::false_type{}, 0u);
    }
    __builtin_amdgcn_s_setprio(1);
    wave_sync();
}

// The same channels from global memory (a FED larger than the stage), as digi words: one lane per
// channel expands its runs, four ADC bytes per iteration.
template <int W, int DW, int S>
__device__ __forceinline__ void build_words(TileSmem<W, DW, S>& sm, uint32_t w, uint32_t* dl,
                                            gconst<uint8_t>* src, uint32_t c0, uint32_t c1) {
    const uint32_t b0 = digi_base(sm, c0 + w);
    for (uint32_t ch = c0 + lane(); ch < c1; ch += kWave) {
        const uint32_t bw = sm.ch_base[ch + w];
        if (bw & kChBad) continue;
        const uint32_t p = sm.ch_pos[ch];
        const uint32_t len = payload_len(sm, ch);
        uint32_t o = bw - b0;
        uint32_t q = 0;
        while (q < len) {
            const uint32_t first = src[p + q], cnt = src[p + q + 1];
            const uint32_t base = (ch << 18) | (first << 10);
            const uint32_t s = p + q + 2;
            uint32_t i = 0;
            for (; i + 4 <= cnt; i += 4) {
                const uint32_t a0 = src[s + i], a1 = src[s + i + 1], a2 = src[s + i + 2],
                               a3 = src[s + i + 3];
                dl[o + i] = base + (i << 10) + a0;
                dl[o + i + 1] = base + ((i + 1) << 10) + a1;
                dl[o + i + 2] = base + ((i + 2) << 10) + a2;
                dl[o + i + 3] = base + ((i + 3) << 10) + a3;
            }
            for (; i < cnt; ++i) dl[o + i] = base + (i << 10) + src[s + i];
            o += cnt;
            q += 2 + cnt;
        }
    }
    wave_sync();
}

// Dense rows of channels [c0, c1) -> digi words; 4 channels per wave step, 16 lanes x 16 strips.
template <int W, int DW, int S>
__device__ __forceinline__ void build_dense(TileSmem<W, DW, S>& sm, uint32_t w, uint32_t* dl,
                                            const uint8_t* rows, uint32_t c0, uint32_t c1) {
    const uint32_t b0 = digi_base(sm, c0 + w);
    for (uint32_t cb = c0; cb < c1; cb += 4) {
        const uint32_t ch = cb + (lane() >> 4);
        const uint32_t s0 = (lane() & 15) * 16;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (ch < c1) v = *gc(reinterpret_cast<const u32x4*>(rows + ch * kStripsPerChannel + s0));
        const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
        uint32_t cnt = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) cnt += ((wds[k >> 2] >> ((k & 3) * 8)) & 255u) != 0u;
        uint32_t tot;
        uint32_t o = seg16_excl_scan(cnt, tot);
        if (ch < c1) {
            o += digi_base(sm, ch + w) - b0;
            const uint32_t base = (ch << 18) | (s0 << 10);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const uint32_t a = (wds[k >> 2] >> ((k & 3) * 8)) & 255u;
                if (a) dl[o++] = base + ((uint32_t)k << 10) + a;
            }
        }
    }
    wave_sync();
}

// digi count of one dense channel row (16-byte loads)
__device__ __forceinline__ uint32_t count_dense_row(const uint8_t* row) {
    uint32_t cnt = 0;
    gconst<u32x4>* r4 = gc(reinterpret_cast<const u32x4*>(row));
#pragma unroll 4
    for (int i = 0; i < kStripsPerChannel / 16; ++i) {
        const u32x4 v = r4[i];
        const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            // the top bit of each nonzero byte
            const uint32_t x = wds[k];
            const uint32_t nz = ((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x;
            cnt += __popc(nz & 0x80808080u);
        }
    }
    return cnt;
}

// Bit i: byte i of the 16 is not zero.
__device__ __forceinline__ uint32_t nonzero_bytes(u32x4 v) {
    const uint32_t wds[4] = {v.x, v.y, v.z, v.w};
    uint32_t m = 0;
#pragma unroll
    for (int k = 3; k >= 0; --k) {
        // the top bit of each nonzero byte, then the four next to each other
        const uint32_t x = wds[k];
        uint32_t nz = ((((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) >> 7) & 0x01010101u;
        nz |= nz >> 7;
        nz |= nz >> 14;
        m = m << 4 | (nz & 15u);
    }
    return m;
}

// All digi words of a channel group in one pass over its dense rows: a lane takes 16 strips, a step
// four channels, so lane order is list order and a scan over the lanes places each step's digis.
// Returns their number, or kNoStrip if they do not fit the list (nothing is lost: the group is then
// taken in chunks). The loads of six steps are in flight together. (Rows counted a lane each and then
// read again took 36 us for 440 FEDs with two waves each, this 17 with four; the rows' bytes alone
// take 2 at a copy's rate: bound by one FED's chain of load, scan, passes and look-back.)
template <int W, int DW, int S>
__device__ __forceinline__ uint32_t build_dense_group(TileSmem<W, DW, S>& sm, uint32_t* dl,
                                                      const uint8_t* rows, uint32_t c_lo) {
    constexpr int kBatch = 6, kSteps = kNch / W / 4;
    static_assert(kSteps % kBatch == 0, "whole batches");
    gconst<u32x4>* src = gc(reinterpret_cast<const u32x4*>(rows + c_lo * kStripsPerChannel)) + lane();
    uint32_t n = 0;
    for (int b = 0; b < kSteps; b += kBatch) {
        u32x4 v[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) v[k] = src[(b + k) * kWave];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const uint32_t wds[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
            uint32_t m = nonzero_bytes(v[k]), tot;
            uint32_t o = n + wave_excl_scan(__popc(m), tot);
            n += tot;
            if (n > (uint32_t)DW) return kNoStrip;   // uniform
            const uint32_t base = (c_lo * kStripsPerChannel + ((uint32_t)(b + k) * kWave + lane()) * 16u) << 10;
            while (m) {
                const uint32_t i = (uint32_t)__builtin_ctz(m);
                m &= m - 1u;
                const uint32_t lo = i & 4u ? wds[1] : wds[0], hi = i & 4u ? wds[3] : wds[2];
                const uint32_t a = ((i & 8u ? hi : lo) >> ((i & 3u) * 8u)) & 255u;
                dl[o++] = base + (i << 10) + a;
            }
        }
    }
    wave_sync();
    return n;
}

// ---- windows of the digi list ---------------------------------------------------------------
// Forming and writing take the list in windows of up to 256 digis, four consecutive ones per lane
// (lane l: slots 4 l .. 4 l + 3 of the window). A window begins where a run can begin and is cut
// where the last run of its 256 slots may begin, so that no run crosses from one window to the
// next; a channel has 256 strips, so a window always holds the run it begins with (in a module
// row, whose runs may have 768 strips, a run that fills its window is taken one digi at a time).
// What a run is follows from wave masks, one per slot of a lane: they are combined by scalar
// instructions, which cost the vector units nothing. Sums go along the four digis of a lane in
// order, then from lane to lane, once per further lane of the longest run (mostly once).
// Bound by vector instruction issue. Two digis per lane with six-step lane scans of every sum, as
// before, took 8758 vector instructions per tile of a 64-event batch (440 FEDs, 0.5 to 5 %
// occupancy) and 0.471 ms for the launch, the windows 5551 and 0.376 ms (with what has been
// shortened since, 3951 and 0.279). Four per lane rather than more: a wave's share of a FED is 370
// to 1700 digis, and a window costs the same however few it holds.
constexpr uint32_t kWindow = 4 * kWave;

// The last slot whose mask bit is set (at least one is).
__device__ __forceinline__ uint32_t last_slot(const uint64_t (&m)[4]) {
    const uint64_t any = m[0] | m[1] | m[2] | m[3];
    const uint32_t l = 63u - (uint32_t)__builtin_clzll(any);
    const uint64_t bit = 1ull << l;
    return 4u * l + ((m[3] & bit) ? 3u : (m[2] & bit) ? 2u : (m[1] & bit) ? 1u : 0u);
}

// Slots [0, n) of a window, as masks.
__device__ __forceinline__ uint64_t slots_below(uint32_t k, uint32_t n) {
    return __ballot(4u * lane() + k < n);
}

// The four words of each lane from slot base on; past nd they read as 0. (Reads at most three
// words past nd: the list's pad.)
__device__ __forceinline__ void read_words(const uint32_t* dl, uint32_t base, uint32_t nd,
                                           uint32_t (&v)[4]) {
    const uint32_t l4 = 4u * lane(), m = nd - base;
    const uint32_t* at = dl + base + (l4 < m ? l4 : m - 1u);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = at[k];
    if (m < kWindow) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = l4 + k < m ? v[k] : 0u;
    }
}

struct Window {
    uint32_t base, n;     // first slot and digis taken; n = 0: a module-row chain longer than this
    uint32_t raw[4];      // the list's words
    uint32_t pos4[4];     // position << 2
    uint32_t adc[4];
    float noise[4];
    uint64_t head[4];     // digis that do not follow the one before them on the adjacent strip
};

// Whether the digi at pos4 goes on from one at prev4 on the strip before it, in the same channel
// or module row.
template <bool kMod>
__device__ __forceinline__ bool follows(uint32_t pos4, uint32_t prev4, Joins J) {
    bool in_row = (pos4 & (255u << 2)) != 0u;
    if constexpr (kMod) in_row = in_row || joined(J, pos4 >> 10);
    return in_row && pos4 == prev4 + 4u;
}

// The window at base: markers become positions and ADCs (kMarkers; else the list holds words), the
// window is cut, and its noise loads are issued.
template <bool kMod, bool kMarkers>
__device__ __forceinline__ Window load_window(const uint32_t* dl, uint32_t base, uint32_t nd,
                                              const uint8_t* stage, gconst<float>* noise, Joins J,
                                              bool maybe) {
    Window x;
    x.base = base;
    read_words(dl, base, nd, x.raw);
    const uint32_t m = nd - base;
    if constexpr (kMarkers) {
        // the largest marker at or before each slot (digi words are below every marker)
        uint32_t s[4];
        s[0] = x.raw[0];
#pragma unroll
        for (int k = 1; k < 4; ++k) s[k] = __builtin_elementwise_max(s[k - 1], x.raw[k]);
        const uint32_t before = from_prev_lane(wave_incl_max(s[3]));
        const uint32_t j0 = (base + 4u * lane()) * kSlotStep;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t t = __builtin_elementwise_max(s[k], before) + j0 + (uint32_t)k * kSlotStep;
            x.pos4[k] = t & kNoiseMask;
            x.adc[k] = stage[(t >> 17) & 0x3fffu];
            x.head[k] = __ballot((int32_t)x.raw[k] < 0);
        }
        if (maybe) {   // uniform
            const uint32_t prev = from_prev_lane(x.pos4[3]);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                bool on = (x.raw[k] & kMaybeBit) != 0u;
                if constexpr (kMod) on = on && follows<kMod>(x.pos4[k], k ? x.pos4[k ? k - 1 : 0] : prev, J);
                x.head[k] &= ~__ballot(on);
            }
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x.pos4[k] = (x.raw[k] >> 8) & kNoiseMask;
            x.adc[k] = x.raw[k] & 255u;
        }
        const uint32_t prev = from_prev_lane(x.pos4[3]);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            x.head[k] = __ballot(!follows<kMod>(x.pos4[k], k ? x.pos4[k ? k - 1 : 0] : prev, J));
    }
    x.head[0] |= 1ull;   // where a window begins, a run can begin
    x.n = m;
    if (m > kWindow) {
        x.n = last_slot(x.head);
        if (x.n == 0u) x.n = kMod ? 0u : kWindow;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        x.noise[k] = *reinterpret_cast<gconst<float>*>(reinterpret_cast<gconst<uint8_t>*>(noise) + x.pos4[k]);
    return x;
}

// ---- cluster forming --------------------------------------------------------------------------
// The cluster threshold, exactly (§2: charge against the cluster threshold): (float)Q >= t *
// sqrtf(S), S = fmaf(n, n, S) from the run's first strip, both roots and products rounded once.
__device__ __forceinline__ bool passes_exactly(float q, float S, float t) {
    return q >= t * __builtin_sqrtf(S);
}

// Runs of one window; puts the words of its clusters' members down from slot n_adc on and counts its
// clusters and member ADCs (uniform; n_adc counts from the list's start). A member's slot is at or
// below its own, and later windows are read from slots above all of these.
// Only members are kept: of the strips above twice their noise that a front end sends, many
// belong to no cluster (46 % of the digis at 1.5 % occupancy, 37 % over 0.5 to 5 %), and the writes
// take that many windows less. 64 events of 440 FEDs: 306 -> 283 us, 64 busy ones 690 -> 641.
//  * cluster threshold: the sums S and Q are the definition's own (S in strip order), and the test
//    q >= t sqrt(S) is taken on squares first: q q >= S t2_hi passes and q q < S t2_lo fails, with
//    t2_hi and t2_lo = t^2 (1 +- 2^-19). Every rounding on either way is 2^-24 or less relative
//    (three here, twice two in the definition's own test), so what the squares decide the
//    definition decides the same; the few runs in between, and any with a NaN, take it exactly.
//    (The host makes the factors NaN where t^2 could leave the normal range.) No root is taken:
//    v_sqrt_f32 runs at a quarter rate, and four slots would need it per lane.
//  * members: a run's digis learn its acceptance from its last one, backwards: through the four
//    slots of a lane mask by mask, and through lanes that one run fills by a carry chain (an
//    addition on the bit-reversed masks).
template <bool kMod>
__device__ __forceinline__ void form_window(uint32_t* dl, const Window& x, const DeviceCalib& cal,
                                            uint32_t& n_cl, uint32_t& n_adc) {
    uint64_t act[4], K[5];   // K: continues the digi before it (both active)
    uint32_t Q[4];                     // raw ADC sum | seed count << kQShift, along the run so far
    float S[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float a = (float)x.adc[k];
        act[k] = __ballot(a > cal.t_channel * x.noise[k]) & slots_below(k, x.n);
        const bool seed = a > cal.t_seed * x.noise[k];
        Q[k] = seed ? x.adc[k] | 1u << kQShift<kMod> : x.adc[k];
    }
    K[0] = act[0] & (act[3] << 1) & ~x.head[0];
#pragma unroll
    for (int k = 1; k < 4; ++k) K[k] = act[k] & act[k - 1] & ~x.head[k];
    K[4] = K[0] >> 1;   // the next lane's first digi continues slot 3
    S[0] = x.noise[0] * x.noise[0];
#pragma unroll
    for (int k = 1; k < 4; ++k) {
        S[k] = __builtin_fmaf(x.noise[k], x.noise[k], in_mask(K[k]) ? S[k - 1] : 0.0f);
        Q[k] += in_mask(K[k]) ? Q[k - 1] : 0u;
    }
    if (K[0]) {   // runs that go on from the lane before
        const uint64_t through = K[0] & K[1] & K[2] & K[3];
        uint64_t deep = K[0];   // lanes whose run began at least so many lanes before
        uint32_t cq = 0u, out = Q[3];
        do {
            const float cs = __uint_as_float(from_prev_lane(__float_as_uint(S[3])));
            S[0] = __builtin_fmaf(x.noise[0], x.noise[0], in_mask(K[0]) ? cs : 0.0f);
#pragma unroll
            for (int k = 1; k < 4; ++k)
                S[k] = __builtin_fmaf(x.noise[k], x.noise[k], in_mask(K[k]) ? S[k - 1] : 0.0f);
            const uint32_t prev = from_prev_lane(out);
            cq = in_mask(K[0]) ? prev : 0u;
            out = Q[3] + (in_mask(through) ? cq : 0u);
            deep = K[0] & ((through & deep) << 1);
        } while (deep);
        Q[0] += cq;
        Q[1] += in_mask(K[1]) ? cq : 0u;
        Q[2] += in_mask(K[1] & K[2]) ? cq : 0u;
        Q[3] += in_mask(K[1] & K[2] & K[3]) ? cq : 0u;
    }
    uint64_t yes[4], open[4];
    float q[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        q[k] = (float)(Q[k] & ((1u << kQShift<kMod>) - 1u));
        const float q2 = q[k] * q[k];
        const uint64_t ends = act[k] & ~K[k + 1] & __ballot(Q[k] >= 1u << kQShift<kMod>);
        const uint64_t above = __ballot(q2 >= S[k] * cal.t2_hi);
        yes[k] = ends & above;
        open[k] = ends & ~above & ~__ballot(q2 < S[k] * cal.t2_lo);
    }
    if (open[0] | open[1] | open[2] | open[3]) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            yes[k] |= open[k] & __ballot(passes_exactly(q[k], S[k], cal.t_cluster));
    }
    // slot 0 of each lane: accepted if its run ends in the lane and was accepted there, or goes
    // through it to an accepted one
    const uint64_t past = K[1] & K[2] & K[3] & K[4];
    uint64_t first = yes[0] | (K[1] & (yes[1] | (K[2] & (yes[2] | (K[3] & yes[3])))));
    if (past) {
        const uint64_t p = __builtin_bitreverse64(past), r = __builtin_bitreverse64(first);
        const uint64_t s = (r << 1) & p;
        first = __builtin_bitreverse64(r | (p & (~(p + s) | s)));
    }
    uint64_t mem[4];
    mem[3] = yes[3] | (K[4] & (first >> 1));
    mem[2] = yes[2] | (K[3] & mem[3]);
    mem[1] = yes[1] | (K[2] & mem[2]);
    mem[0] = yes[0] | (K[1] & mem[1]);
    uint32_t o = n_adc;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        n_cl += popc(yes[k]);
        n_adc += popc(mem[k]);
        o = count_below(mem[k], o);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t word = x.pos4[k] << 8 | x.adc[k] | (in_mask(K[k]) ? kContBit : 0u);
        if (in_mask(mem[k])) dl[o] = word;
        o += in_mask(mem[k]) ? 1u : 0u;
    }
}

// A chain of adjacent digis that fills the window at base (module rows only), one digi at a time,
// the same in every lane; returns the slot after it. (n_cl, n_adc and the members' slots as in
// form_window)
template <bool kMarkers>
__device__ uint32_t form_long_chain(uint32_t* dl, uint32_t base, uint32_t nd, const uint8_t* stage,
                                    gconst<float>* noise, Joins J, const DeviceCalib& cal,
                                    uint32_t& n_cl, uint32_t& n_adc) {
    uint32_t marker = 0u, prev4 = 0u, j = base, head = base, Q = 0u, seeds = 0u;
    float S = 0.0f;
    bool open = false;
    auto close = [&](uint32_t end) {   // the run [head, end)
        if (open && seeds && passes_exactly((float)Q, S, cal.t_cluster)) {
            n_cl += 1u;
            for (uint32_t i = head; i < end; ++i)
                dl[n_adc++] = uni(dl[i]) | (i > head ? kContBit : 0u);
        }
        open = false;
    };
    for (; j < nd; ++j) {
        const uint32_t raw = uni(dl[j]);
        uint32_t pos4, adc;
        if constexpr (kMarkers) {
            if (raw & kMarker) marker = raw;
            const uint32_t t = marker + j * kSlotStep;
            pos4 = t & kNoiseMask;
            adc = uni(stage[(t >> 17) & 0x3fffu]);
        } else {
            pos4 = (raw >> 8) & kNoiseMask;
            adc = raw & 255u;
        }
        if (j > base && !follows<true>(pos4, prev4, J)) break;
        prev4 = pos4;
        const float n = __uint_as_float(uni(__float_as_uint(noise[pos4 >> 2])));
        const float a = (float)adc;
        if (a > cal.t_channel * n) {
            if (!open) {
                open = true;
                head = j;
                Q = seeds = 0u;
                S = 0.0f;
            }
            Q += adc;
            seeds += a > cal.t_seed * n ? 1u : 0u;
            S = __builtin_fmaf(n, n, S);
        } else {
            close(j);
        }
        dl[j] = pos4 << 8 | adc;
    }
    close(j);
    return j;
}

// Forming over the digi list dl[0, nd) of a FED, the next window's loads in flight (without module
// rows). The list becomes that of the n_adc members.
template <bool kMod, bool kMarkers>
__device__ __forceinline__ void form_pass(uint32_t* dl, uint32_t nd, const uint8_t* stage,
                                          const DeviceCalib& cal, uint32_t fed, Joins J, bool maybe,
                                          uint32_t& n_cl, uint32_t& n_adc) {
    gconst<float>* noise = gc(cal.noise) + fed * kStripsPerFed;
    uint32_t ncl = 0, nadc = 0, base = 0;
    auto load = [&](uint32_t at) {
        return load_window<kMod, kMarkers>(dl, at, nd, stage, noise, J, maybe);
    };
    if (nd) {
        Window x = load(0u);
        for (;;) {
            if constexpr (kMod) {
                if (x.n == 0u) {
                    base = form_long_chain<kMarkers>(dl, x.base, nd, stage, noise, J, cal, ncl, nadc);
                    if (base >= nd) break;
                    x = load(base);
                    continue;
                }
            }
            base = x.base + x.n;
            if (base >= nd) {
                form_window<kMod>(dl, x, cal, ncl, nadc);
                break;
            }
            if constexpr (kMod) {   // (the registers do not reach for two windows)
                form_window<kMod>(dl, x, cal, ncl, nadc);
                x = load(base);
            } else {
                const Window next = load(base);
                form_window<kMod>(dl, x, cal, ncl, nadc);
                x = next;
            }
        }
    }
    n_cl = ncl;
    n_adc = nadc;
    wave_sync();
}

// ---- outputs ------------------------------------------------------------------------------
// The float nearest to N / D for integers 0 <= N < 2^53 and 0 < D < 2^27, the same float as
// (float)(N / D) with the double quotient. One Newton step takes the hardware reciprocal
// estimate (good to 2^-14 or better) to y within 2^-28 of 1/D. The remainder r = N - D q1 of
// q1 = N y is exact (a multiple of ulp(q1), fewer than 2^28 of them), and q2 = q1 + r y =
// N/D + (q1 - N/D)(1 - D y), rounded, lies within 2^-53 + 2^-55 relative of N / D. A quotient
// that is not a float midpoint lies at least 2^-25 / D > 2^-52 relative from one (it differs
// from it by a multiple of the midpoint's last bit over D), so q2 rounds to the same float; a
// midpoint is a double, and q2 is that double.
__device__ __forceinline__ float quotient_to_float(double N, double D) {
    const double y0 = __builtin_amdgcn_rcp(D);
    const double y = __builtin_fma(y0, __builtin_fma(-D, y0, 1.0), y0);
    const double q1 = N * y;
    const double r = __builtin_fma(-D, q1, N);
    return (float)__builtin_fma(r, y, q1);
}

// A cluster's record from its last digi dw: rp = its width - 1, C the charge, M the sum of strip * c.
// Module rows: the cluster may start in an earlier channel of the row, so its channel and first
// strip come from the position of its first digi (d_pos(dw) - rp), and the strip moment from that
// channel's strip 0 is sum(pos * c) - 256 ch C, with sum(pos * c) = 4096 Mh + M (pos * c < 2^31,
// summed in two parts so that 768 strips cannot overflow: M < 768 x 2^12 < 2^22, Mh < 768 x 2^19).
template <bool kMod>
__device__ __forceinline__ u32x4 make_record(uint32_t fed, uint32_t dw, uint32_t rp, uint32_t C,
                                             uint32_t M, uint32_t Mh) {
    uint32_t ch, first;
    double m;
    if constexpr (kMod) {
        const uint32_t head = d_pos(dw) - rp;
        ch = head >> 8;
        first = head & 255u;
        m = ((double)Mh * 4096.0 + (double)M) - 256.0 * (double)ch * (double)C;   // exact
    } else {
        ch = d_ch(dw);
        first = d_strip(dw) - rp;
        m = (double)M;
    }
    const uint32_t width = rp + 1u;
    // barycenter: sum (s+1/2) c / sum c = (2M + C) / (2C), numerator and denominator exact
    // integers (2C < 2^27: C <= 768 x 65535). Both forms are computed, so that no branch splits
    // the window; the quotient is not used when C = 0.
    const float q = quotient_to_float(2.0 * m + (double)C, 2.0 * (double)C);
    const float mid = (float)first + (float)width * 0.5f;
    const float bary = C ? q : mid;
    return u32x4{fed * kNch + ch, first | (width << 16), C, __float_as_uint(bary)};
}

// Gain-corrected ADC min(rint(a / g), 65535) with the FP32 quotient, g and r = its reciprocal
// rounded to nearest. regular: every usable gain of the detector lies in [2^-60, 2^60]; then a r
// is within an ulp of a / g, the remainder of one fmaf is exact, and the corrected quotient is
// the correctly rounded one (Markstein, "Computation of elementary functions on the IBM RISC
// System/6000 processor", 1990): three instructions for the division's ten.
__device__ __forceinline__ uint32_t corrected_adc(uint32_t adc, float g, float r, bool regular) {
    const float a = (float)adc;
    const float q0 = a * r;
    float q = __builtin_fmaf(__builtin_fmaf(-q0, g, a), r, q0);
    if (!regular) {   // uniform; the empty asm keeps the division from being taken in any case
        asm volatile("");
        q = a / g;
    }
    return (uint32_t)__builtin_fminf(__builtin_rintf(q), 65535.0f);
}

// The sums of a run, carried from lane to lane: v[i][k] holds the sums along the digis of the lane
// up to slot k, and gets what the lanes before hold of slot 0's run. K as in form_window.
template <int N>
__device__ __forceinline__ void carry_sums(uint32_t (&v)[N][4], const uint64_t (&K)[5]) {
    if (!K[0]) return;
    const uint64_t through = K[0] & K[1] & K[2] & K[3];
    uint64_t deep = K[0];
    uint32_t c[N], out[N];
#pragma unroll
    for (int i = 0; i < N; ++i) out[i] = v[i][3];
    do {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t prev = from_prev_lane(out[i]);
            c[i] = in_mask(K[0]) ? prev : 0u;
            out[i] = v[i][3] + (in_mask(through) ? c[i] : 0u);
        }
        deep = K[0] & ((through & deep) << 1);
    } while (deep);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        v[i][0] += c[i];
        v[i][1] += in_mask(K[1]) ? c[i] : 0u;
        v[i][2] += in_mask(K[1] & K[2]) ? c[i] : 0u;
        v[i][3] += in_mask(K[1] & K[2] & K[3]) ? c[i] : 0u;
    }
}

// A cluster that fills its window (module rows only), one member at a time, the same in every
// lane; returns the slot after it.
template <int W, int DW, int S>
__device__ uint32_t write_long_cluster(const TileSmem<W, DW, S>& sm, const uint32_t* dl,
                                       uint32_t base, uint32_t nd, uint32_t fed,
                                       const EventDesc& ev, bool regular, uint32_t& rc,
                                       uint32_t& pa) {
    gmut<uint16_t>* adc_out = gm(ev.adc);
    uint32_t C = 0u, M = 0u, Mh = 0u, last = 0u, j = base;
    for (; j < nd; ++j) {
        const uint32_t d = uni(dl[j]);
        if (j > base && d < kContBit) break;
        const float* gr = sm.gain + 2u * (d_pos(d) >> 7);
        const uint32_t c = uni(corrected_adc(d_adc(d), gr[0], gr[1], regular));
        const uint32_t m = d_pos(d) * c;
        C += c;
        M += m & 0xfffu;
        Mh += m >> 12;
        if (pa < ev.cap_adc) adc_out[pa] = (uint16_t)c;
        ++pa;
        last = d;
    }
    const u32x4 rec = make_record<true>(fed, last, j - base - 1u, C, M, Mh);
    if (rc < ev.cap_cl) gm(reinterpret_cast<u32x4*>(ev.cl))[rc] = rec;
    ++rc;
    return j;
}

// Records and member ADCs of the formed list dl[0, nd) at their final positions, by windows as in
// forming (here cut at the last digi that continues no cluster). The member ADCs are
// gain-corrected here; a lane's four lie together and leave in one 8-byte store (of any 2-byte
// alignment). Straight-line windows: every value of a window is formed first and the
// stores come last, so that no lane mask has to live across a branch.
template <bool kMod, int W, int DW, int S>
__device__ __forceinline__ void write_pass(const TileSmem<W, DW, S>& sm, const uint32_t* dl,
                                           uint32_t nd, uint32_t fed, const EventDesc& ev,
                                           bool regular, uint32_t base_cl, uint32_t base_adc) {
    gmut<uint16_t>* adc_out = gm(ev.adc);
    gmut<u32x4>* cl_out = gm(reinterpret_cast<u32x4*>(ev.cl));
    uint32_t rc = base_cl, pa = base_adc;
    for (uint32_t base = 0; base < nd;) {
        uint32_t d[4];
        read_words(dl, base, nd, d);
        uint64_t valid[4], K[5];   // K: continues the cluster of the one before
#pragma unroll
        for (int k = 0; k < 4; ++k) K[k] = __ballot(d[k] >= kContBit);
        uint32_t n = nd - base;
        if (n > kWindow) {
            const uint64_t heads[4] = {~K[0] | 1ull, ~K[1], ~K[2], ~K[3]};
            n = last_slot(heads);
            if (n == 0u) {
                if constexpr (kMod) {
                    base = write_long_cluster(sm, dl, base, nd, fed, ev, regular, rc, pa);
                    continue;
                }
                n = kWindow;
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            valid[k] = slots_below(k, n);
            K[k] &= valid[k];
        }
        base += n;
        K[4] = K[0] >> 1;
        // corrected ADCs, and the sums along clusters: charge, strip moment and width
        uint32_t c[4], s[4];
        constexpr int kSums = kMod ? 3 : 2;   // C | width << 24, M; module rows: C, M | width << 22, Mh
        uint32_t v[kSums][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float* gr = sm.gain + ((d[k] >> 16) & 0x1feu);   // 2 x (position / 128)
            c[k] = corrected_adc(d_adc(d[k]), gr[0], gr[1], regular);
            s[k] = d_strip(d[k]);
            const bool on = k && in_mask(K[k]);
            if constexpr (kMod) {
                const uint32_t m = __umul24(d_pos(d[k]), c[k]);
                v[0][k] = c[k] + (on ? v[0][k ? k - 1 : 0] : 0u);
                v[1][k] = (m & 0xfffu) + (1u << 22) + (on ? v[1][k ? k - 1 : 0] : 0u);
                v[2][k] = (m >> 12) + (on ? v[2][k ? k - 1 : 0] : 0u);
            } else {
                // at most 256 x 65535 < 2^24; a width of 256 reads as 0
                v[0][k] = c[k] + (1u << 24) + (on ? v[0][k ? k - 1 : 0] : 0u);
                v[1][k] = mad24(s[k], c[k], on ? v[1][k ? k - 1 : 0] : 0u);
            }
        }
        carry_sums(v, K);
        // positions: records by their cluster's last digi
        uint64_t end[4];
        uint32_t rr[4];
        rr[0] = rc;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            end[k] = valid[k] & ~K[k + 1];
            rr[0] = count_below(end[k], rr[0]);
            rc += popc(end[k]);
        }
#pragma unroll
        for (int k = 1; k < 4; ++k) rr[k] = rr[k - 1] + (in_mask(end[k - 1]) ? 1u : 0u);
        // Records by pairs of digis A and B: at most one cluster of the pair has more than one
        // member, and rec1 is A's where it ends at A, else B's. Where A's cluster ends at A, one
        // that ends at B is B alone: first = its strip, width 1, barycenter strip + 1/2 exactly
        // (the quotient (2 s c + c) / (2 c), and the midpoint when c = 0), in a module row too
        // (its channel is its own); that record is formed without the division.
        u32x4 rec1[2], rec2[2];
        uint64_t any[2], both[2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int A = 2 * p, B = A + 1;
            const bool eA = in_mask(end[A]);
            const uint32_t dw = eA ? d[A] : d[B];
            const uint32_t v0 = eA ? v[0][A] : v[0][B], v1 = eA ? v[1][A] : v[1][B];
            if constexpr (kMod) {
                const uint32_t v2 = eA ? v[2][A] : v[2][B];
                rec1[p] = make_record<true>(fed, dw, (v1 >> 22) - 1u, v0, v1 & 0x3fffffu, v2);
            } else {
                rec1[p] = make_record<false>(fed, dw, ((v0 >> 24) - 1u) & 255u, v0 & 0xffffffu, v1, 0u);
            }
            rec2[p] = u32x4{fed * kNch + d_ch(d[B]), s[B] | (1u << 16), c[B],
                            __float_as_uint((float)s[B] + 0.5f)};
            any[p] = end[A] | end[B];
            both[p] = end[A] & end[B];
        }
        // (uniform: mostly the whole window fits)
        const uint32_t room = pa < ev.cap_adc ? ev.cap_adc - pa : 0u, n_out = n < room ? n : room;
        if (rc > ev.cap_cl) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                any[p] &= __ballot(rr[2 * p] < ev.cap_cl);
                both[p] &= __ballot(rr[2 * p + 1] < ev.cap_cl);
            }
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if (in_mask(any[p])) *at_offset(cl_out, 16u * rr[2 * p]) = rec1[p];
            if (in_mask(both[p])) *at_offset(cl_out, 16u * rr[2 * p + 1]) = rec2[p];
        }
        const uint32_t l4 = 4u * lane();
        gmut<uint16_t>* at = at_offset(adc_out, 2u * (pa + l4));
        const u32x2 c4{c[0] | c[1] << 16, c[2] | c[3] << 16};
        if (l4 + 4u <= n_out) {
            *reinterpret_cast<gmut<u32x2_by2>*>(at) = c4;
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (l4 + k < n_out) at[k] = (uint16_t)c[k];
        }
        pa += n;
    }
    wave_sync();
}

// ---- decoupled look-back over the FEDs of one event -----------------------------------------
// A FED's counts are published as soon as they are known; look_back sums those of the FEDs before
// it: lane i reads the word of FED top-i, so 64 predecessors are inspected per load; only words not
// yet published are waited for. Only the counts travel through these words, so relaxed atomics
// suffice. All values steering the loop are uniform.
__device__ __forceinline__ void publish(unsigned long long* row, uint32_t f, uint32_t n_cl,
                                        uint32_t n_adc) {
    __hip_atomic_store(&row[f], pack_state(f == 0u ? kFlagIncl : kFlagAgg, n_cl, n_adc),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// (resumable: run() looks at most `polls` times and returns whether it is done)
struct LookBack {
    int top;              // highest FED not yet summed
    uint32_t cl, adc;     // sums of the FEDs above it
    uint32_t polls_left;  // the wait bound
    bool done, failed;
    __device__ __forceinline__ void start(uint32_t f) {
        top = (int)f - 1;
        cl = adc = 0u;
        polls_left = kSpinLimit;
        done = f == 0u;
        failed = false;
    }
    __device__ __forceinline__ void run(const unsigned long long* row, uint32_t polls) {
        while (!done && polls) {
            const int k = top - (int)lane();
            unsigned long long v = pack_state(kFlagIncl, 0u, 0u);   // before FED 0: nothing
            if (k >= 0) v = __hip_atomic_load(&row[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t flag = (uint32_t)(v >> 62);
            const uint64_t incl = __ballot(flag == kFlagIncl);
            const uint64_t none = __ballot(flag == 0u);
            const uint32_t first_incl = incl ? (uint32_t)__builtin_ctzll(incl) : 64u;
            const uint32_t first_none = none ? (uint32_t)__builtin_ctzll(none) : 64u;
            // lanes summed now: up to the first inclusive word, stopping before any unpublished
            const uint32_t n_take = first_none <= first_incl ? first_none : first_incl + 1u;
            const bool take = lane() < n_take;
            cl += wave_sum(take ? (uint32_t)((v >> 31) & 0x7fffffffu) : 0u);
            adc += wave_sum(take ? (uint32_t)(v & 0x7fffffffu) : 0u);
            done = first_incl < first_none;          // reached an inclusive word
            top -= (int)n_take;
            if (!done && first_none < 64u) {         // FED `top` has not published yet
                if (--polls_left == 0u) { failed = done = true; break; }
                --polls;
                __builtin_amdgcn_s_sleep(2);
            }
        }
    }
};

// A word of an event's result in host memory.
__device__ __forceinline__ void store_result(uint32_t* word, uint32_t v) {
    __hip_atomic_store(word, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Whether an event has a malformed channel among a wave's, and the channels' status bits where the
// event wants them.
template <int W, int DW, int S>
__device__ __forceinline__ void emit_status(const TileSmem<W, DW, S>& sm, uint32_t w, uint32_t c_lo,
                                            uint32_t c_hi, bool any_bad, uint32_t trailing,
                                            uint8_t* chan_status, uint32_t f, EventResult* res) {
    if (chan_status) {   // uniform
        for (uint32_t ch = c_lo + lane(); ch < c_hi; ch += kWave)
            gm(chan_status)[f * kNch + ch] =
                (uint8_t)(((sm.ch_base[ch + w] & kChBad) ? (uint32_t)SC_CH_MALFORMED : 0u) |
                          (trailing ? (uint32_t)SC_CH_FED_TRAILING : 0u));
    }
    if (any_bad) store_result(&res->malformed, 1u);   // uniform; the same store from every lane
}

// What a wave knows of its formed channel group.
struct Group {
    uint32_t n_cl, n_adc;             // clusters and member ADCs of its chunks
    uint32_t last_cl, last_adc;       // of the last chunk, which stays in the digi list
};
// The FED's counts and what lies before a wave's group in it.
struct FedCounts {
    uint32_t n_cl, n_adc, pre_cl, pre_adc;
    bool chunked;   // some group has more than one chunk: they are built again for their writes
};

// Counts of one channel group, one pass over each of its chunks (shared by the ZS and the dense
// front ends). form(c0, c1, nd, n_cl, n_adc) fills the group's digi list with channels [c0, c1), nd
// digis, forms it and counts its clusters and member ADCs.
template <int W, int DW, int S, class FormFn>
__device__ __forceinline__ Group form_group(TileSmem<W, DW, S>& sm, uint32_t w, uint32_t n_chunks,
                                            FormFn form) {
    const uint8_t* cf = sm.chunk_first[w];
    Group g{};
    for (uint32_t ci = 0; ci < n_chunks; ++ci) {
        const uint32_t c0 = uni(cf[ci]), c1 = uni(cf[ci + 1]);
        const uint32_t nd = uni(digi_base(sm, c1 + w) - digi_base(sm, c0 + w));
        form(c0, c1, nd, g.last_cl, g.last_adc);
        g.n_cl += g.last_cl;
        g.n_adc += g.last_adc;
    }
    return g;
}

// The waves of a tile exchange their groups' counts in LDS (a barrier of the tile: the digi lists
// are formed and the stage is free after it, unless some group is chunked).
template <int W, int DW, int S>
__device__ __forceinline__ FedCounts exchange_counts(TileSmem<W, DW, S>& sm, uint32_t w,
                                                     const Group& g, uint32_t n_chunks) {
    sm.grp_cnt[w][0] = g.n_cl;   // uniform values from every lane
    sm.grp_cnt[w][1] = g.n_adc;
    sm.grp_cnt[w][2] = n_chunks;
    tile_sync();
    FedCounts r{};
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)W; ++i) {
        const uint32_t c = uni(sm.grp_cnt[i][0]), a = uni(sm.grp_cnt[i][1]);
        r.pre_cl += i < w ? c : 0u;
        r.pre_adc += i < w ? a : 0u;
        r.n_cl += c;
        r.n_adc += a;
        r.chunked |= uni(sm.grp_cnt[i][2]) > 1u;
    }
    return r;
}

// The rest of one wave's look-back for the FED, its offsets left in LDS for all waves, the event's
// results.
template <int W, int DW, int S>
__device__ __forceinline__ void resolve_offsets(const FusedArgs& A, TileSmem<W, DW, S>& sm,
                                                uint32_t e, uint32_t f, const FedCounts& n,
                                                LookBack& lb) {
    const uint32_t n_fed = A.cal.n_fed;
    unsigned long long* row = A.tile_state + (size_t)e * n_fed;
    lb.run(row, 0xffffffffu);
    if (f)
        __hip_atomic_store(&row[f], pack_state(kFlagIncl, lb.cl + n.n_cl, lb.adc + n.n_adc),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sm.grp_cnt[W][0] = lb.cl;
    sm.grp_cnt[W][1] = lb.adc;
    // uniform branches; every lane stores the same values
    if (lb.failed) store_result(&A.res[e].failed, 1u);
    if (f == n_fed - 1) {
        store_result(&A.res[e].n_cl, lb.cl + n.n_cl);
        store_result(&A.res[e].n_adc, lb.adc + n.n_adc);
    }
}

// What the writes need of an event.
__device__ __forceinline__ EventDesc event_outputs(const FusedArgs& A, uint32_t e) {
    const EventDesc* evp = A.ev + e;
    EventDesc ev{};
    ev.cl = uniptr(evp->cl);
    ev.adc = uniptr(evp->adc);
    ev.cap_cl = uni(evp->cap_cl);
    ev.cap_adc = uni(evp->cap_adc);
    return ev;
}

// Writes of a wave's digi list (the last chunk of its group) at its offset: the FED's (from LDS),
// the groups before it and the chunks before it.
template <int W, int DW, bool kMod, int S>
__device__ __forceinline__ void write_list(const FusedArgs& A, TileSmem<W, DW, S>& sm,
                                           const EventDesc& ev, uint32_t f, uint32_t w,
                                           const Group& g, const FedCounts& n) {
    write_pass<kMod>(sm, sm.digi + w * TileSmem<W, DW, S>::kList, g.last_adc, f, ev,
                     A.cal.regular_gains != 0u,
                     uni(sm.grp_cnt[W][0]) + n.pre_cl + g.n_cl - g.last_cl,
                     uni(sm.grp_cnt[W][1]) + n.pre_adc + g.n_adc - g.last_adc);
}

// The earlier chunks of a chunked group, built and formed again.
template <int W, int DW, bool kMod, int S, class FormFn>
__device__ __forceinline__ void write_chunks(const FusedArgs& A, TileSmem<W, DW, S>& sm,
                                             const EventDesc& ev, uint32_t f, uint32_t w, const FedCounts& n,
                                             uint32_t n_chunks, FormFn form) {
    const uint32_t* dl = sm.digi + w * TileSmem<W, DW, S>::kList;
    const uint8_t* cf = sm.chunk_first[w];
    uint32_t oc = uni(sm.grp_cnt[W][0]) + n.pre_cl, oa = uni(sm.grp_cnt[W][1]) + n.pre_adc;
    for (uint32_t ci = 0; ci + 1 < n_chunks; ++ci) {
        const uint32_t c0 = uni(cf[ci]), c1 = uni(cf[ci + 1]);
        const uint32_t nd = uni(digi_base(sm, c1 + w) - digi_base(sm, c0 + w));
        uint32_t ccl, cadc;
        form(c0, c1, nd, ccl, cadc);
        write_pass<kMod>(sm, dl, cadc, f, ev, A.cal.regular_gains != 0u, oc, oa);
        oc += ccl;
        oa += cadc;
    }
}

// Channel group of wave w: [c_lo, c_hi).
template <int W>
__device__ __forceinline__ void group_range(uint32_t w, uint32_t& c_lo, uint32_t& c_hi) {
    c_lo = w * (uint32_t)(kNch / W);
    c_hi = c_lo + (uint32_t)(kNch / W);
}

// ---- one (event, FED) tile from ZS bytes --------------------------------------------------
// The FED's join words (module rows), uniform.
template <bool kMod>
__device__ __forceinline__ Joins fed_joins(const DeviceCalib& cal, uint32_t f) {
    if constexpr (kMod) {
        gconst<uint32_t>* j = gc(cal.joins) + 4u * f;
        return Joins{uni(j[0]), uni(j[1]), uni(j[2])};
    } else {
        return Joins{0u, 0u, 0u};
    }
}

// A tile as event and FED (e = kNoTile: none left).
struct Ticket {
    uint32_t e, f;
};

// t / n for n = A.n_ev, with ev_magic = ceil(2^32 / n) (0 stands for n = 1): the high half of the
// product is the quotient or one more.
__device__ __forceinline__ uint32_t div_events(const FusedArgs& A, uint32_t t) {
    if (A.ev_magic == 0u) return t;   // uniform
    const uint32_t q = __umulhi(t, A.ev_magic);
    return q * A.n_ev > t ? q - 1u : q;
}

// A tile of the launch: FED f of event e, L bytes at g.
struct Tile {
    uint32_t e, f, L;
    const uint8_t* g;
    __device__ __forceinline__ bool none() const { return e == kNoTile; }
};

// A ticket's tile, looked up and left in LDS for all waves (by one wave).
template <int W, int DW, int S>
__device__ __forceinline__ void post_tile(const FusedArgs& A, TileSmem<W, DW, S>& sm,
                                          const Ticket& t) {
    uint32_t L = 0u;
    uint64_t g = 0u;
    if (t.e != kNoTile) {   // uniform
        gconst<uint64_t>* off = gc(uniptr(A.ev[t.e].fed_off)) + t.f;
        const uint64_t lo = uni64(off[0]), hi = uni64(off[1]);
        L = hi > lo ? (uint32_t)(hi - lo) : 0u;
        g = reinterpret_cast<uint64_t>(uniptr(A.ev[t.e].zs)) + lo;
    }
    sm.next[0] = t.e;
    sm.next[1] = t.f;
    sm.next[2] = L;
    sm.next[3] = (uint32_t)g;
    sm.next[4] = (uint32_t)(g >> 32);
}
template <int W, int DW, int S>
__device__ __forceinline__ Tile posted_tile(const TileSmem<W, DW, S>& sm) {
    return Tile{uni(sm.next[0]), uni(sm.next[1]), uni(sm.next[2]),
                reinterpret_cast<const uint8_t*>((uint64_t)uni(sm.next[3]) | (uint64_t)uni(sm.next[4]) << 32)};
}

// The tiles that a workgroup takes, the writes of each after the first half of the next. A tile's
// look-back waits for the FEDs before it that are still being formed, so the offsets are asked for
// late: once a tile's digi lists are formed and its counts published, the stage is free, and the
// next tile is taken, staged, walked and checked before the offsets are needed and the lists
// written; then its own lists are built. The writes need the digi lists and the gains only; each
// wave replaces the gains of its own channels after them.
// A ticket is not taken earlier than that: the tile behind it would begin late, by as much as the
// one before it is large, and every later FED of its event would wait for it (with tickets taken
// one tile ahead and the bytes under way meanwhile the waits grew from 6k to 43k cycles per tile).
// A tile with a chunked group builds it again from the stage for its writes: those come first.
// The waits end because a workgroup that waits for a tile's offsets holds no unformed tile before it
// in its queue's order: of the waiting tiles take the first; what it waits for lies before it, so it
// is not held up by another waiting one. Tiles of another queue (order 2) can be of lower FEDs, and
// are taken only when the writes of the last of this one are done (other()).
// Issue priorities (s_setprio): 3 in the walk, which a tile's other waves wait for, 2 in the other
// phases that mostly wait for memory or LDS (ticket, staging, check, markers), 1 in forming, whose
// counts later FEDs wait for, 0 in the writes: 64 ordinary events of 440 FEDs 288 -> 279 us, 64 busy
// ones 642 -> 613, 13 with module rows 119 -> 110, 20 events and single ones the same. The ticket's
// atomic beside the exchange: 20 events 96 -> 94 us, 64 busy ones 618 -> 613, module rows 109 -> 110.
// The offsets asked for late: 64 events of 440 FEDs waited 2.9k cycles per tile for them instead of
// 6.3k, most of which the other phases took up (vector issue is 70 % busy); one event: 30.3 -> 27.5 us.
template <int W, int DW, bool kMod, int S, class FirstFn, class AskFn, class TakeFn, class OtherFn>
__device__ __forceinline__ void run_zs_tiles(const FusedArgs& A, TileSmem<W, DW, S>& sm,
                                             FirstFn first, AskFn ask, TakeFn take,
                                             OtherFn other) {
    const uint32_t w = wave_index<W>();
    const bool lead = w == 0u, last = w == (uint32_t)W - 1u;
    uint32_t c_lo, c_hi;
    group_range<W>(w, c_lo, c_hi);
    uint32_t* dl = sm.digi + w * TileSmem<W, DW, S>::kList;
    // the tile before, whose writes are due (p.none(): none)
    Tile p{kNoTile, 0u, 0u, nullptr};
    Group p_grp{};
    FedCounts p_cnt{};
    LookBack lb{};
    if (last) post_tile(A, sm, first());
    tile_sync();
    bool more = true;
    for (;;) {
        const Tile t = more ? posted_tile(sm) : Tile{kNoTile, 0u, 0u, nullptr};
        uint32_t n_chunks = 0;
        bool any_bad = false, any_on = false;
        GainVecs<W> gains;
        WalkResult wk{};
        Joins J{};
        gconst<uint8_t>* gg = gc(t.g);
        if (!t.none()) {   // uniform over the tile's waves
            load_gains(gains, A.cal.gain, t.f, w);
            if (fits_stage(sm, t.L)) {
                Pieces<S, kWave * W> bytes;
                bytes.load(t.g, t.L, threadIdx.x);
                bytes.store(sm.stage, t.g, t.L, threadIdx.x);
                tile_sync();
            }
            if (lead) walk_fed(sm, t.g, t.L);
            if (W > 1 && last && !p.none())
                lb.run(A.tile_state + (size_t)p.e * A.cal.n_fed, kWalkPolls);
            tile_sync();
            wk = walk_result(sm, t.L);
            J = fed_joins<kMod>(A.cal, t.f);
            if (wk.fits) {
                const uint8_t* st = sm.stage;
                n_chunks = plan_chunks<kMod>(sm, w, c_lo, c_hi, J,
                                             [&](uint32_t ch, bool on, uint32_t& near) {
                                                 return check_channel(sm, st, ch, wk, on, near);
                                             },
                                             any_bad, any_on);
            } else {
                n_chunks = plan_chunks<kMod>(sm, w, c_lo, c_hi, J,
                                             [&](uint32_t ch, bool on, uint32_t& near) {
                                                 return check_channel(sm, gg, ch, wk, on, near);
                                             },
                                             any_bad, any_on);
            }
            emit_status(sm, w, c_lo, c_hi, any_bad, wk.trailing,
                        A.any_status ? uniptr(A.ev[t.e].chan_status) : nullptr, t.f,
                        A.res + t.e);
        }
        if (!p.none()) {
            const EventDesc ev = event_outputs(A, p.e);
            if (last) resolve_offsets(A, sm, p.e, p.f, p_cnt, lb);
            tile_sync();
            __builtin_amdgcn_s_setprio(0);
            write_list<W, DW, kMod>(A, sm, ev, p.f, w, p_grp, p_cnt);
        }
        if (t.none()) {
            if (!more) break;
            p.e = kNoTile;
            tile_sync();   // (every wave has read the posted tile)
            if (last) post_tile(A, sm, other());
            tile_sync();
            more = !posted_tile(sm).none();
            if (!more) break;
            continue;
        }
        store_gains(sm, gains, w);
        auto form = [&](uint32_t c0, uint32_t c1, uint32_t nd, uint32_t& n_cl, uint32_t& n_adc) {
            if (wk.fits) {
                build_markers<kMod>(sm, w, dl, J, any_on, c0, c1);
                form_pass<kMod, true>(dl, nd, sm.stage, A.cal, t.f, J, any_on, n_cl, n_adc);
            } else {
                build_words(sm, w, dl, gg, c0, c1);
                form_pass<kMod, false>(dl, nd, sm.stage, A.cal, t.f, J, false, n_cl, n_adc);
            }
        };
        p_grp = form_group(sm, w, n_chunks, form);
        more = !A.one_each;   // uniform over the grid: no second tile
        const uint32_t asked = last && more ? ask() : kNoTile;   // (the next tile's ticket)
        p_cnt = exchange_counts(sm, w, p_grp, n_chunks);
        __builtin_amdgcn_s_setprio(2);
        p = t;
        if (last) publish(A.tile_state + (size_t)t.e * A.cal.n_fed, t.f, p_cnt.n_cl, p_cnt.n_adc);
        lb.start(t.f);
        if (p_cnt.chunked) {   // uniform over the tile's waves
            const EventDesc ev = event_outputs(A, p.e);
            if (last) resolve_offsets(A, sm, p.e, p.f, p_cnt, lb);
            tile_sync();
            write_list<W, DW, kMod>(A, sm, ev, p.f, w, p_grp, p_cnt);
            write_chunks<W, DW, kMod>(A, sm, ev, p.f, w, p_cnt, n_chunks, form);
            p.e = kNoTile;
        }
        if (more) {
            if (last) post_tile(A, sm, take(asked));
            tile_sync();   // (every wave is done with the stage)
        }
    }
}

// ---- one FED tile from dense ADC rows (single event) --------------------------------------
template <int W, int DW, bool kMod, int S>
__device__ void dense_tile(const FusedArgs& A, TileSmem<W, DW, S>& sm, const uint8_t* dense,
                           uint32_t f) {
    const uint8_t* rows = dense + (size_t)f * kStripsPerFed;
    const uint32_t w = wave_index<W>();
    GainVecs<W> gains;
    load_gains(gains, A.cal.gain, f, w);
    store_gains(sm, gains, w);
    uint32_t c_lo, c_hi;
    group_range<W>(w, c_lo, c_hi);
    const Joins J = fed_joins<kMod>(A.cal, f);
    uint32_t* dl = sm.digi + w * TileSmem<W, DW, S>::kList;
    const uint32_t n_digis = build_dense_group(sm, dl, rows, c_lo);
    const bool whole = n_digis != kNoStrip;   // uniform
    uint32_t n_chunks = 1u;
    if (whole) {
        sm.ch_base[c_lo + w] = 0u;
        sm.ch_base[c_hi + w] = (uint16_t)n_digis;
        sm.chunk_first[w][0] = (uint8_t)c_lo;
        sm.chunk_first[w][1] = (uint8_t)c_hi;
        wave_sync();
    } else {
        bool any_bad, any_on;
        n_chunks = plan_chunks<kMod>(
            sm, w, c_lo, c_hi, J,
            [&](uint32_t ch, bool, uint32_t&) { return count_dense_row(rows + ch * kStripsPerChannel); },
            any_bad, any_on);
    }
    auto form = [&](uint32_t c0, uint32_t c1, uint32_t nd, uint32_t& n_cl, uint32_t& n_adc) {
        if (!whole) build_dense(sm, w, dl, rows, c0, c1);
        form_pass<kMod, false>(dl, nd, sm.stage, A.cal, f, J, false, n_cl, n_adc);
    };
    const Group grp = form_group(sm, w, n_chunks, form);
    const FedCounts cnt = exchange_counts(sm, w, grp, n_chunks);
    const EventDesc ev = event_outputs(A, 0u);
    if (w == 0u) {
        publish(A.tile_state, f, cnt.n_cl, cnt.n_adc);
        LookBack lb;
        lb.start(f);
        resolve_offsets(A, sm, 0u, f, cnt, lb);
    }
    tile_sync();
    write_list<W, DW, kMod>(A, sm, ev, f, w, grp, cnt);
    write_chunks<W, DW, kMod>(A, sm, ev, f, w, cnt, n_chunks, form);
}

// ---- kernels --------------------------------------------------------------------------------
// Orders 0 and 1: the next ticket of the one queue (by one wave). Every lane executes the atomic,
// adding 1 from lane 0 and 0 from the others (no lane test); lane 0's old value is the ticket.
// Tiles are taken in a global order (event-major or FED-major) in which a tile's look-back
// predecessors come before it, so the lowest unfinished tile of an event has always been taken and
// every look-back ends, whatever part of the grid is resident.
__device__ __forceinline__ Ticket claim_one(const FusedArgs& A) {
    const uint32_t n_fed = A.cal.n_fed;
    const uint32_t t = uni(atomicAdd(A.queue, lane() == 0u ? 1u : 0u));
    if (t >= A.n_ev * n_fed) return Ticket{kNoTile, 0u};
    if (A.fed_major) {
        const uint32_t f = div_events(A, t);
        return Ticket{t - f * A.n_ev, f};
    }
    const uint32_t e = t / n_fed;
    return Ticket{e, t - e * n_fed};
}

// Tile order 2: G = 8 queues (one in a grid of fewer workgroups); queue x holds the FEDs f = x
// (mod G), FED-major, its tickets counted in queue[x * kQueueStride] (one cache line each). A
// workgroup's home queue is blockIdx mod G. In a launch with a workgroup for every tile (one_each) it
// takes its own place there (blockIdx / G), without an atomic: as many workgroups asking at once
// for a ticket cost such a launch 2 us. Its look-backs wait for workgroups of lower index only, which
// start first. (Places for the first tiles of larger launches would hang where a grid is not resident
// as a whole: tiles taken later would wait for places whose workgroups cannot start.)
// Else a workgroup takes tickets from its home until that is
// exhausted, then, with none of its tiles' writes left, moves on to another open queue; it ends once
// every queue is known to be exhausted.
// Look-back ends here too, if the whole grid is resident (the host launches this order only
// with no other such launch running, and never with more workgroups than fit): take the unfinished
// tile of lowest FED. Either it has been taken, and its predecessors (lower FEDs) are finished,
// or it is still in its queue x; then queue x is not exhausted, so the workgroups of home x (at
// least one, resident) hold only tiles of queue x taken before it, of FED at most its own,
// which finish and take it next.
struct XcdCursor {
    uint32_t cur;     // the queue claimed from
    uint32_t known;   // bit x: queue x is exhausted (a ticket past its end, or its counter seen so)
};

__device__ __forceinline__ uint32_t queue_shift() { return gridDim.x < kXcds ? 0u : kXcdShift; }

// Tiles of queue x.
__device__ __forceinline__ uint32_t queue_tiles(const FusedArgs& A, uint32_t x) {
    const uint32_t s = queue_shift(), n_fed = A.cal.n_fed;
    return x < n_fed ? ((n_fed - x + (1u << s) - 1u) >> s) * A.n_ev : 0u;
}
__device__ __forceinline__ Ticket tile_of(const FusedArgs& A, uint32_t x, uint32_t t) {
    const uint32_t j = div_events(A, t);
    return Ticket{t - j * A.n_ev, x + (j << queue_shift())};
}

__device__ __forceinline__ Ticket claim_xcd(const FusedArgs& A, XcdCursor& c) {
    const uint32_t groups = 1u << queue_shift(), all = (1u << groups) - 1u;
    // each pass either returns a tile or adds a queue to `known`: at most groups + 1 passes
    for (uint32_t k = 0; k <= groups && c.known != all; ++k) {
        const uint32_t x = uni(c.cur);   // a scalar address: one atomic per wave, not per lane
        const uint32_t size = queue_tiles(A, x);
        if (size && !(c.known >> x & 1u)) {
            const uint32_t t = uni(atomicAdd(A.queue + x * kQueueStride, lane() == 0u ? 1u : 0u));
            if (t < size) return tile_of(A, x, t);
        }
        c.known |= 1u << x;
        // the next queue not known to be exhausted, from the counters (lane i reads queue i's);
        // a counter only grows, so one read at or past the end is final, and a stale lower read
        // costs one more failed ticket
        bool open = false;
        if (lane() < groups && !(c.known >> lane() & 1u)) {
            const uint32_t v = __hip_atomic_load(A.queue + lane() * kQueueStride, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
            open = v < queue_tiles(A, lane());
        }
        const uint32_t m = (uint32_t)__ballot(open);
        c.known = uni(c.known | (all & ~m));
        if (!m) break;
        const uint32_t after = m & ~((2u << x) - 1u);   // open queues past x, then from 0
        c.cur = uni((uint32_t)__builtin_ctz(after ? after : m));
    }
    return Ticket{kNoTile, 0u};
}

// The same in two halves, so that the atomic is under way while the caller does something else: the
// home queue's (or the present one's) ticket asked for, its answer not looked at, ...
__device__ __forceinline__ uint32_t ask_xcd(const FusedArgs& A, const XcdCursor& c) {
    const uint32_t x = uni(c.cur);
    if (c.known >> x & 1u) return kNoTile;
    return atomicAdd(A.queue + x * kQueueStride, lane() == 0u ? 1u : 0u);
}
// ... and the tile it stands for (none: that queue is exhausted).
__device__ __forceinline__ Ticket take_xcd(const FusedArgs& A, XcdCursor& c, uint32_t asked) {
    const uint32_t x = uni(c.cur), a = uni(asked);
    if (a != kNoTile && a < queue_tiles(A, x)) return tile_of(A, x, a);
    c.known |= 1u << x;
    return Ticket{kNoTile, 0u};
}

// A workgroup's first tile: a ticket, or its own place in its home queue (none if that is past the
// queue's end: the homes have the same number of workgroups, the queues not always of tiles).
__device__ __forceinline__ Ticket first_xcd(const FusedArgs& A, XcdCursor& c) {
    if (!A.one_each) return claim_xcd(A, c);
    const uint32_t s = queue_shift();
    const uint32_t x = blockIdx.x & ((1u << s) - 1u), t = blockIdx.x >> s;
    return t < queue_tiles(A, x) ? tile_of(A, x, t) : Ticket{kNoTile, 0u};
}

// Whether the events are for the large shape: runs of four FEDs per sampled tile, the same ones for
// every wave. It is for launches with a FED past the small stage among them (1 of 256 stands for about
// 0.4 %; the shapes cross between 0.05 and 0.5 %), or with one in eight a long one.
__device__ __forceinline__ bool for_large_shape(const FusedArgs& A) {
    static_assert(kSmallStageFed == (uint32_t)kStageSmall - 16u, "what the small stage holds");
    const uint32_t shift = sampled_shift(A.n_ev), n_fed = A.cal.n_fed;
    uint32_t longs = 0u;
    bool past = false;
    for (uint32_t r = 0; r < 1u << shift; ++r) {
        const SampledTile t = sampled_tile(r * kWave + lane(), shift, A.n_ev, n_fed);
        gconst<uint64_t>* off = gc(gc(A.ev)[t.e].fed_off);
        uint64_t at[kSampledRun + 1];
#pragma unroll
        for (uint32_t i = 0; i <= kSampledRun; ++i) at[i] = off[t.f + i < n_fed ? t.f + i : n_fed];
#pragma unroll
        for (uint32_t i = 0; i < kSampledRun; ++i) {
            const uint64_t L = at[i + 1] > at[i] ? at[i + 1] - at[i] : 0u;
            past |= L > kSmallStageFed;
            longs += L >= kLongFed ? 1u : 0u;
        }
    }
    const uint32_t n = kSampledRun * kWave << shift;
    return sc::for_large_shape(popc(__ballot(past)), n, wave_sum(longs), n);
}

// Whether this launch is the one that runs, where two are enqueued for the same events. The first one
// leaves its answer for the second, which reads a word where it would begin with two dependent loads.
__device__ __forceinline__ bool picked(const FusedArgs& A) {
    if (A.pick == 1u) return gc(A.queue)[kPickedWord] == 0u;
    const bool large = for_large_shape(A);
    if (blockIdx.x == 0u) gm(A.queue)[kPickedWord] = large ? 1u : 0u;
    return large;
}

// At most 128 vector registers for tiles of two and four waves, so that the eight and four tiles that
// fit a CU's LDS can be resident (four waves per SIMD). (64 busy events with the large shape take 765
// us with 130 registers, 620 with 128.)
constexpr int min_waves_per_simd(int w) { return w == 1 ? 1 : 4; }

template <int W, int DW, bool kMod, int S>
__global__ __launch_bounds__(kWave * W, min_waves_per_simd(W)) void fused_kernel(FusedArgs A) {
    __shared__ TileSmem<W, DW, S> sm;
    if (A.pick && !picked(A)) return;   // uniform over the grid
    XcdCursor cur{blockIdx.x & ((1u << queue_shift()) - 1u), 0u};
    run_zs_tiles<W, DW, kMod>(
        A, sm, [&]() { return A.fed_major == 2u ? first_xcd(A, cur) : claim_one(A); },
        [&]() { return A.fed_major == 2u ? ask_xcd(A, cur) : kNoTile; },
        [&](uint32_t asked) { return A.fed_major == 2u ? take_xcd(A, cur, asked) : claim_one(A); },
        [&]() { return A.fed_major == 2u && !A.one_each ? claim_xcd(A, cur) : Ticket{kNoTile, 0u}; });
}

template <int W, int DW, bool kMod, int S>
__global__ __launch_bounds__(kWave * W, min_waves_per_simd(W)) void cluster_dense_kernel(const uint8_t* dense, FusedArgs A) {
    __shared__ TileSmem<W, DW, S> sm;
    for (;;) {
        if (wave_index<W>() == 0u) {
            const Ticket t = claim_one(A);   // n_ev = 1, FED-major
            sm.next[0] = t.e;
            sm.next[1] = t.f;
        }
        tile_sync();
        const uint32_t f = uni(sm.next[1]);
        if (uni(sm.next[0]) == kNoTile) break;
        dense_tile<W, DW, kMod>(A, sm, dense, f);
        tile_sync();   // the tile ends here for every lane of every wave (a convergent point)
    }
}

// ZS -> dense rows, a workgroup of four waves per FED: the stage, the walk, then a lane per channel
// checks its records and expands them into zeroed rows in LDS, which all threads copy out with 16-byte
// stores. Bound by its chains (the walk's 96 LDS round trips, a channel's records); one wave per FED
// with 16 channels at a time took 49 us for 440 FEDs, this 17 us.
constexpr int kUnpackWaves = 4;
constexpr uint32_t kRowStride = kStripsPerChannel + 16;   // the lanes' rows start at different banks

// One valid channel's records into its zeroed row. (staged: up to three bytes past a record are read)
template <class P>
__device__ __forceinline__ void expand_channel(P src, uint32_t a, uint32_t end, uint8_t* row) {
    constexpr bool kStaged = std::is_same_v<P, const uint8_t*>;
    while (a < end) {
        const uint32_t first = src[a], cnt = src[a + 1u];
        a += 2u;
        uint8_t* out = row + first;
        if constexpr (kStaged) {
            for (uint32_t i = 0; i < cnt; i += 4u) {
                const uint8_t b0 = src[a + i], b1 = src[a + i + 1u], b2 = src[a + i + 2u],
                              b3 = src[a + i + 3u];
                out[i] = b0;
                if (i + 1u < cnt) out[i + 1u] = b1;
                if (i + 2u < cnt) out[i + 2u] = b2;
                if (i + 3u < cnt) out[i + 3u] = b3;
            }
        } else {
            for (uint32_t i = 0; i < cnt; ++i) out[i] = src[a + i];
        }
        a += cnt;
    }
}

__global__ __launch_bounds__(kWave * kUnpackWaves) void unpack_kernel(
    const uint8_t* zs, const uint64_t* fed_off, uint8_t* dense, uint8_t* chan_status,
    EventResult* res) {
    constexpr int W = kUnpackWaves, S = kStageLarge;
    __shared__ TileSmem<W, 4, S> sm;
    __shared__ alignas(16) uint8_t rows[kNch * kRowStride + 16];
    const uint32_t f = blockIdx.x, w = wave_index<W>();
    const uint64_t lo = uni64(gc(fed_off)[f]), hi = uni64(gc(fed_off)[f + 1]);
    const uint32_t L = hi > lo ? (uint32_t)(hi - lo) : 0u;
    const uint8_t* g = zs + lo;
    Pieces<S, kWave * W> bytes;
    if (fits_stage(sm, L)) bytes.load(g, L, threadIdx.x);
    u32x4* row4 = reinterpret_cast<u32x4*>(rows);
    for (uint32_t i = threadIdx.x; i < kNch * kRowStride / 16u; i += kWave * W)
        row4[i] = u32x4{0u, 0u, 0u, 0u};
    if (fits_stage(sm, L)) bytes.store(sm.stage, g, L, threadIdx.x);
    tile_sync();
    if (w == 0u) walk_fed(sm, g, L);
    tile_sync();
    const WalkResult wk = walk_result(sm, L);
    bool bad = false;
    if (lane() < (uint32_t)(kNch / W)) {
        const uint32_t ch = w * (uint32_t)(kNch / W) + lane();
        uint8_t* row = rows + ch * kRowStride;
        uint32_t near;
        if (wk.fits) {
            const uint8_t* s = sm.stage;
            bad = check_channel(sm, s, ch, wk, false, near) == kChBad;
            if (!bad) expand_channel(s, sm.ch_pos[ch], sm.ch_pos[ch] + payload_len(sm, ch), row);
        } else {
            gconst<uint8_t>* s = gc(g);
            bad = check_channel(sm, s, ch, wk, false, near) == kChBad;
            if (!bad) expand_channel(s, sm.ch_pos[ch], sm.ch_pos[ch] + payload_len(sm, ch), row);
        }
        if (chan_status)
            gm(chan_status)[f * kNch + ch] = (uint8_t)((bad ? (uint32_t)SC_CH_MALFORMED : 0u) |
                                                       (wk.trailing ? (uint32_t)SC_CH_FED_TRAILING : 0u));
    }
    if (__ballot(bad)) store_result(&res->malformed, 1u);
    tile_sync();
    constexpr uint32_t kRowVecs = kStripsPerChannel / 16;
    gmut<u32x4>* out = gm(reinterpret_cast<u32x4*>(dense + (size_t)f * kStripsPerFed));
#pragma unroll
    for (uint32_t i = threadIdx.x; i < kNch * kRowVecs; i += kWave * W)
        out[i] = row4[i / kRowVecs * (kRowStride / 16u) + i % kRowVecs];
}

__global__ void reset_kernel(unsigned long long* state, uint32_t n_state, uint32_t* queue) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t k = i; k < n_state; k += stride) state[k] = 0ull;
    if (i < kXcds) queue[i * kQueueStride] = 0u;
}

// Effective noise per strip: the noise itself, or +inf when the strip is unusable (bad flag,
// noise NaN / negative / infinite, APV gain NaN / <= 0), so that ADC > T*noise never holds
// for it (T >= 0 finite: T*inf is +inf, or NaN for T = 0; both compare false).
// gain_pairs: each APV's gain and its reciprocal, rounded to nearest.
__global__ void derive_calib_kernel(const float* noise, const float* gain, const uint8_t* bad,
                                    uint32_t n_strips, float* out, float* gain_pairs) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_strips) return;
    if (i < n_strips / kStripsPerApv) {
        gain_pairs[2 * i] = gain[i];
        gain_pairs[2 * i + 1] = 1.0f / gain[i];
    }
    const float n = noise[i];
    const float g = gain[i / kStripsPerApv];
    const bool usable = bad[i] == 0 && !__builtin_isnan(n) && n >= 0.0f && !__builtin_isinf(n) &&
                        !__builtin_isnan(g) && g > 0.0f;
    out[i] = usable ? n : __builtin_inff();
}

// Resident tiles per CU of a kernel (its LDS and registers), queried once per shape.
template <int W, int DW, bool kMod, int S>
int blocks_per_cu_for(bool dense) {
    static std::atomic<int> known[2] = {0, 0};
    int nb = known[dense].load(std::memory_order_relaxed);
    if (nb > 0) return nb;
    hipError_t e = dense ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, cluster_dense_kernel<W, DW, kMod, S>, kWave * W, 0)
                         : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fused_kernel<W, DW, kMod, S>, kWave * W, 0);
    if (e != hipSuccess || nb < 1) return 1;
    // (LDS is given out in pieces of 1280 bytes, which that count may take for smaller ones: it said 12
    // for single-wave tiles of 13008 bytes, of which a CU holds 11)
    constexpr size_t lds = (sizeof(TileSmem<W, DW, S>) + 1279) / 1280 * 1280;
    nb = std::min(nb, (int)(160 * 1024 / lds));
    known[dense].store(nb, std::memory_order_relaxed);
    return nb;
}

// Module rows need a whole row (up to 768 digis) in one chunk of a wave's list.
constexpr int kRowDigis = 3 * kStripsPerChannel;

// Tile shapes: W waves per tile, chunk_digis digis per tile (chunk_digis / W per wave) and the
// stage size; the large stage exists for four shapes. stage 0 means the small one.
template <class F>
bool dispatch(uint32_t w, uint32_t d, uint32_t stage, F&& f) {
    if (stage == 0u) stage = (uint32_t)kStageSmall;
#define SC_CASE(WW, DD, SS) \
    if (w == WW && d == DD && stage == (uint32_t)SS) { \
        f(std::integral_constant<int, WW>{}, std::integral_constant<int, DD / WW>{}, \
          std::integral_constant<int, SS>{}); \
        return true; \
    }
    SC_CASE(1, 1024, kStageSmall) SC_CASE(1, 2048, kStageSmall) SC_CASE(1, 3072, kStageSmall)
    SC_CASE(1, 4096, kStageSmall)
    SC_CASE(2, 2048, kStageSmall) SC_CASE(2, 2880, kStageSmall) SC_CASE(2, 3072, kStageSmall)
    SC_CASE(2, 4096, kStageSmall)
    SC_CASE(4, 2048, kStageSmall) SC_CASE(4, 3072, kStageSmall) SC_CASE(4, 4096, kStageSmall)
    SC_CASE(2, 2048, kStageLarge) SC_CASE(2, 2880, kStageLarge) SC_CASE(4, 4096, kStageLarge)
    SC_CASE(4, 6144, kStageLarge)
#undef SC_CASE
    return false;
}

}  // namespace

bool tile_shape_supported(uint32_t waves, uint32_t d, uint32_t stage) {
    return dispatch(waves, d, stage, [](auto, auto, auto) {});
}

bool tile_shape_supports_modules(uint32_t waves, uint32_t d) {
    bool ok = false;
    auto rows = [&](auto, auto DW, auto) { ok = decltype(DW)::value >= kRowDigis; };
    if (!dispatch(waves, d, 0u, rows)) dispatch(waves, d, (uint32_t)kStageLarge, rows);
    return ok;
}

uint32_t stage_bytes_of(uint32_t stage) { return stage ? stage : (uint32_t)kStageSmall; }

// The dense front end never reads the stage: it runs with the small one where the shape has it.
uint32_t dense_stage(uint32_t waves, uint32_t d, uint32_t stage) {
    return tile_shape_supported(waves, d, 0u) ? 0u : stage;
}

int fused_blocks_per_cu(uint32_t waves, uint32_t d, bool dense, bool modules, uint32_t stage) {
    int nb = 1;
    dispatch(waves, d, dense ? dense_stage(waves, d, stage) : stage, [&](auto W, auto DW, auto SS) {
        constexpr int w = decltype(W)::value, dw = decltype(DW)::value, st = decltype(SS)::value;
        if constexpr (dw >= kRowDigis) {
            nb = modules ? blocks_per_cu_for<w, dw, true, st>(dense)
                         : blocks_per_cu_for<w, dw, false, st>(dense);
        } else {
            nb = blocks_per_cu_for<w, dw, false, st>(dense);
        }
    });
    return nb;
}

hipError_t launch_derive_calib(const float* noise, const float* gain, const uint8_t* bad,
                               uint32_t n_fed, float* out, float* gain_pairs, hipStream_t stream) {
    const uint32_t n = n_fed * kStripsPerFed;
    (void)hipGetLastError();
    hipLaunchKernelGGL(derive_calib_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, noise,
                       gain, bad, n, out, gain_pairs);
    return hipGetLastError();
}

hipError_t launch_reset(const FusedArgs& a, uint32_t n_state, hipStream_t stream) {
    uint32_t blocks = (n_state + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 1024) blocks = 1024;
    (void)hipGetLastError();
    hipLaunchKernelGGL(reset_kernel, dim3(blocks), dim3(256), 0, stream, a.tile_state, n_state,
                       a.queue);
    return hipGetLastError();
}

// The fused kernel of a shape (NULL: there is none). The module-row kernels (cal.joins set) exist for
// the shapes whose wave lists hold a row.
static const void* fused_function(const FusedArgs& a, uint32_t waves, uint32_t d, uint32_t stage) {
    const bool mod = a.cal.joins != nullptr;
    const void* fn = nullptr;
    dispatch(waves, d, stage, [&](auto W, auto DW, auto SS) {
        constexpr int w = decltype(W)::value, dw = decltype(DW)::value, st = decltype(SS)::value;
        if (!mod) fn = reinterpret_cast<const void*>(&fused_kernel<w, dw, false, st>);
        if constexpr (dw >= kRowDigis)
            if (mod) fn = reinterpret_cast<const void*>(&fused_kernel<w, dw, true, st>);
    });
    return fn;
}

hipError_t launch_fused(const FusedArgs& a, uint32_t waves, uint32_t d, uint32_t stage,
                        uint32_t grid, hipStream_t stream) {
    const void* fn = fused_function(a, waves, d, stage);
    if (!fn) return hipErrorInvalidValue;
    FusedArgs args = a;
    void* params[] = {&args};
    (void)hipGetLastError();
    return hipLaunchKernel(fn, dim3(grid), dim3(kWave * waves), params, 0, stream);
}

hipError_t add_fused(hipGraph_t graph, hipGraphNode_t* last, const FusedArgs& a, uint32_t waves,
                     uint32_t d, uint32_t stage, uint32_t grid) {
    const void* fn = fused_function(a, waves, d, stage);
    if (!fn) return hipErrorInvalidValue;
    FusedArgs args = a;
    void* params[] = {&args};
    hipKernelNodeParams p{};
    p.func = const_cast<void*>(fn);
    p.gridDim = dim3(grid);
    p.blockDim = dim3(kWave * waves);
    p.kernelParams = params;   // (copied by the call)
    hipGraphNode_t node;
    const hipError_t e = hipGraphAddKernelNode(&node, graph, last, *last ? 1 : 0, &p);
    if (e == hipSuccess) *last = node;
    return e;
}

hipError_t launch_cluster_dense(const uint8_t* dense, const FusedArgs& a, uint32_t waves,
                                uint32_t d, uint32_t stage, uint32_t grid, hipStream_t stream) {
    (void)hipGetLastError();
    const bool mod = a.cal.joins != nullptr;
    bool ok = false;
    dispatch(waves, d, dense_stage(waves, d, stage), [&](auto W, auto DW, auto SS) {
        constexpr int w = decltype(W)::value, dw = decltype(DW)::value, st = decltype(SS)::value;
        if constexpr (dw >= kRowDigis) {
            if (mod) hipLaunchKernelGGL((cluster_dense_kernel<w, dw, true, st>), dim3(grid), dim3(kWave * w), 0, stream, dense, a);
            else     hipLaunchKernelGGL((cluster_dense_kernel<w, dw, false, st>), dim3(grid), dim3(kWave * w), 0, stream, dense, a);
            ok = true;
        } else if (!mod) {
            hipLaunchKernelGGL((cluster_dense_kernel<w, dw, false, st>), dim3(grid), dim3(kWave * w), 0, stream, dense, a);
            ok = true;
        }
    });
    return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t launch_unpack(const uint8_t* zs, const uint64_t* fed_off, uint32_t n_fed,
                         uint8_t* dense, uint8_t* chan_status, EventResult* res,
                         hipStream_t stream) {
    (void)hipGetLastError();
    hipLaunchKernelGGL(unpack_kernel, dim3(n_fed), dim3(kWave * kUnpackWaves), 0, stream, zs, fed_off, dense,
                       chan_status, res);
    return hipGetLastError();
}

}  // namespace sc
