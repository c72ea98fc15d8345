// sc_internal.h -- types shared by the HIP kernels and the host runtime of libsc.so.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sc.h"

namespace sc {

constexpr int kChannelsPerFed = 96;
constexpr int kStripsPerChannel = 256;
constexpr int kStripsPerApv = 128;
constexpr int kWave = 64;

// One event of a fused launch, in device memory.
struct EventDesc {
    const uint8_t* zs;          // FED buffers of the event
    const uint64_t* fed_off;    // [n_fed + 1]
    sc_cluster_rec* cl;          // output clusters
    uint16_t* adc;              // output member ADCs
    uint8_t* chan_status;       // optional [n_fed * 96]
    uint32_t cap_cl;
    uint32_t cap_adc;
};

// Per-event result, in pinned host memory that the host clears before the launch: the tile of the
// event's last FED stores the counts, any tile may store 1 to either of the other words (all plain
// stores of one value each, so nothing is read or added across the link).
struct EventResult {
    uint32_t n_cl;
    uint32_t n_adc;
    uint32_t malformed;   // some channel is
    uint32_t failed;      // a look-back gave up waiting
};

// Device-resident calibration, derived once per context.
struct DeviceCalib {
    const float* noise;   // per strip: noise, or +inf when the strip is unusable (kNoisePad more
                          // bytes may be read past the last one)
    const float* gain;    // per APV: gain, 1 / gain
    const uint32_t* joins;   // module rows: [n_fed * 4] words, bit c of word c / 32 of FED f set
                             // when channel c reads the same module as channel c - 1; NULL: none
    uint32_t n_fed;
    float t_seed, t_channel, t_cluster;
    float t2_hi, t2_lo;      // t_cluster^2 (1 +- 2^-19); NaN where the squares decide nothing
    uint32_t regular_gains;  // every usable gain lies in [2^-60, 2^60]
};
// The last window of a FED loads the noise of up to 255 strips past its last digi, unused.
constexpr size_t kNoisePad = 1024;

// Tile ticket counters, one per 128-byte line: counter 0 (orders 0 and 1) or one per XCD
// (order 2, at most 8).
constexpr uint32_t kQueueStride = 32;
constexpr size_t kQueueBytes = 8 * kQueueStride * sizeof(uint32_t);
// Beside counter 0: whether the large shape was picked, for the second of two launches.
constexpr uint32_t kPickedWord = 1;

struct FusedArgs {
    const EventDesc* ev;
    EventResult* res;                // pinned host memory
    unsigned long long* tile_state;  // [n_ev * n_fed] decoupled look-back words
    uint32_t* queue;                 // kQueueBytes of tile ticket counters
    DeviceCalib cal;
    uint32_t n_ev;
    uint32_t fed_major;              // tile order: 0 event-major, 1 FED-major, 2 FED-major per XCD
    uint32_t any_status;             // some event wants its channels' status
    uint32_t ev_magic;               // ceil(2^32 / n_ev), 0 for n_ev = 1
    uint32_t one_each;               // order 2 with a workgroup for every tile: no second tickets
    uint32_t pick;                   // 0: run; of two shapes enqueued for the same events, the large
                                     // one first: 2 look at the FEDs, say so and run if they are for
                                     // it, 1 run if they were not
};
// The FEDs by which a launch's shape is chosen (plan_launches): those past the small stage, which the
// ordinary shape reads from global memory byte by byte while all later FEDs of their event wait, and
// long ones, of whose digis many wave groups have more than the 1440 that its lists hold.
constexpr uint32_t kSmallStageFed = 6640, kLongFed = 6100;
constexpr bool for_large_shape(uint64_t past, uint64_t past_per, uint64_t longs, uint64_t n) {
    return past * past_per >= n || longs * 8u >= n;
}
// Where the workgroups choose by themselves (pick), they look at runs of four FEDs from these tiles on:
// number k of n = 64, 128, 256 or 512. Events and FEDs are spread over the launch each by itself, the
// FEDs in the order of the multiples of 37 modulo n, so that all events (of more, n) and all parts of
// the detector are among them whatever the two counts have in common. (Every n_tiles / 64-th tile in
// FED-major order met one event alone where 64 divides n_fed.)
struct SampledTile {
    uint32_t e, f;
};
constexpr uint32_t kSampledRun = 4;
// log2(n / 64): every event of up to 512 has a run.
constexpr uint32_t sampled_shift(uint32_t n_ev) {
    return n_ev <= 64u ? 0u : n_ev <= 128u ? 1u : n_ev <= 256u ? 2u : 3u;
}
constexpr SampledTile sampled_tile(uint32_t k, uint32_t shift, uint32_t n_ev, uint32_t n_fed) {
    const uint32_t bits = 6u + shift;
    const uint32_t f = (k * 37u & ((1u << bits) - 1u)) * n_fed >> bits;
    const uint32_t last = n_fed > kSampledRun ? n_fed - kSampledRun : 0u;   // a whole run, if there is one
    return SampledTile{(uint32_t)((uint64_t)k * n_ev >> bits), f < last ? f : last};
}

// Scratch of the allocation-free batch call (sc_process_events_static), a file-scope device
// array of sc_kernels.hip: event descriptors, the tile queue and the look-back words, for at most
// SC_STATIC_MAX_EVENTS events and SC_STATIC_MAX_TILES tiles.
constexpr size_t kStaticDescOff = 0;
constexpr size_t kStaticQueueOff = (kStaticDescOff + sizeof(EventDesc) * SC_STATIC_MAX_EVENTS + 255) / 256 * 256;
constexpr size_t kStaticStateOff = kStaticQueueOff + kQueueBytes;
constexpr size_t kStaticScratchBytes = kStaticStateOff + sizeof(unsigned long long) * SC_STATIC_MAX_TILES;
// Device address of that array on the current device (hipGetSymbolAddress; once per device).
hipError_t static_scratch_address(void** ptr);

// Launch helpers (sc_kernels.hip). All enqueue on `stream` and return the launch error.
hipError_t launch_derive_calib(const float* noise, const float* gain, const uint8_t* bad,
                               uint32_t n_fed, float* noise_out, float* gain_pairs,
                               hipStream_t stream);
// Clears n_state look-back words (n_ev x n_fed) and the queue.
hipError_t launch_reset(const FusedArgs& a, uint32_t n_state, hipStream_t stream);
// stage: the LDS stage size in bytes of the tuning (0: the small one)
hipError_t launch_fused(const FusedArgs& a, uint32_t tile_waves, uint32_t chunk_digis,
                        uint32_t stage, uint32_t grid, hipStream_t stream);
// The same launch as a node of a graph, after the node *last (NULL: the first), which it replaces.
hipError_t add_fused(hipGraph_t graph, hipGraphNode_t* last, const FusedArgs& a, uint32_t tile_waves,
                     uint32_t chunk_digis, uint32_t stage, uint32_t grid);
hipError_t launch_cluster_dense(const uint8_t* adc_dense, const FusedArgs& a,
                                uint32_t tile_waves, uint32_t chunk_digis, uint32_t stage,
                                uint32_t grid, hipStream_t stream);
hipError_t launch_unpack(const uint8_t* zs, const uint64_t* fed_off, uint32_t n_fed,
                         uint8_t* adc_dense, uint8_t* chan_status, EventResult* res,
                         hipStream_t stream);
// Cluster -> global hit conversion: per event, its records, their count and its hit output.
struct HitDesc {
    const sc_cluster_rec* cl;
    float* hits;   // 4 floats per cluster
    uint32_t n;
    uint32_t pad;
};
// chan: [n_channels] {module, first module strip}; mod: [2 * n_modules] float4 {origin, pitch},
// {u_dir, module_strips / 2}.
hipError_t launch_hits(const HitDesc* d, uint32_t n_ev, uint32_t max_n, const uint32_t* chan,
                       const float* mod, uint32_t n_channels, hipStream_t stream);

// Resident workgroups per compute unit for a tile shape (waves per tile, digis per chunk, LDS
// stage bytes; 0 is the small stage).
int fused_blocks_per_cu(uint32_t tile_waves, uint32_t chunk_digis, bool dense, bool modules,
                        uint32_t stage);
bool tile_shape_supported(uint32_t tile_waves, uint32_t chunk_digis, uint32_t stage);
// The stage size a tuning's stage value stands for (0: the small one).
uint32_t stage_bytes_of(uint32_t stage);
// Whether a shape's wave lists hold a module row (768 digis): needed while modules are set.
bool tile_shape_supports_modules(uint32_t tile_waves, uint32_t chunk_digis);

}  // namespace sc
