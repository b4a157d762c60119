// swap_kernels.h -- launch interface of the gather/scatter kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "aqua_core.h"

namespace aqua {

struct SwapLaunch {
    bool out;                 // true: pool -> image, false: image -> pool
    uint8_t* pool;            // device pointer of the pool base
    uint8_t* img;             // device-accessible pointer of the buffer base
    uint32_t img_l0;          // layer l's image data starts at img_off + (l - img_l0) * lstride
    const RunDesc* descs;     // device-accessible run descriptors
    const InlineRuns* inl;    // if not null: the runs, passed as a kernel argument instead
    uint32_t ndesc;
    uint32_t first_layer;     // layers [first_layer, first_layer + num_layers)
    uint32_t num_layers;
    uint64_t chunk_bytes;     // C
    uint64_t pool_lstride;    // N * C
    uint64_t mean_run_bytes;  // per layer
    uint64_t max_run_bytes;
    uint32_t max_workgroups;  // 0: as many as part_grid says
    bool nt_pool_store;       // scatter: nontemporal stores into the pool
    bool xcd_units;           // a 1024-lane workgroup per unit instead of a wave per KiB,
                              // and to each XCD a contiguous eighth of the units
};

// Scatter store hint, measured on MI355X.  Nontemporal pool stores pay for
// large chunks and for calls that write much more than the 256 MB last-level
// cache holds.  A smaller call of smaller chunks ends sooner with ordinary
// stores, which L2 and that cache partly absorb:
//   64 KiB chunks: 0-7 % shorter with nontemporal stores, 2 to 10 GiB calls;
//   32 KiB chunks: 10 % longer at 1 GiB per call, 0.5-2 % shorter at 4.4-5 GiB;
//   16 KiB chunks: 20 % longer at 512 MiB per call, 7 % shorter at 2.5 GiB.
// The bytes are the whole call's, also when several launches carry it: ordinary
// stores chosen for each 512 MiB launch of a larger call made its scatter
// 2-15 % longer.
// Runs dealt out to the XCDs turn the smaller calls round: each XCD then
// writes one contiguous stretch of a layer.  Dealt scatters of 2 to 32 KiB
// chunks, nontemporal against ordinary stores: 256 MiB to 1 GiB 10-16 %
// shorter.  Below the 256 MB of the last-level cache it depends on what
// follows: one call after another, 64 MiB 6-10 % and 128 MiB 11-13 % shorter;
// a call by itself, whose stores the cache absorbs, 8-14 % longer (198 MiB 99
// against 86 us).  Those keep ordinary stores.
constexpr uint64_t kNtPoolStoreMinChunk = 64ull << 10;
constexpr uint64_t kNtPoolStoreMinBytes = 2ull << 30;
constexpr uint64_t kNtPoolStoreMinDealt = 256ull << 20;
inline bool nt_pool_store(uint64_t chunk_bytes, uint64_t call_bytes, bool dealt) {
    return chunk_bytes >= kNtPoolStoreMinChunk || call_bytes >= kNtPoolStoreMinBytes ||
           (dealt && call_bytes >= kNtPoolStoreMinDealt);
}

// Enqueues the copy on `stream`; returns the first launch error.  Adds the
// number of kernel launches it made to *launches when that is given.  `done`,
// if given, completes with the last launch: the launch itself carries it
// (hipExtLaunchKernel), or, while the stream is being captured, a record after
// it does.  A record is a packet of its own behind the kernel; measured on
// MI355X, back-to-back calls with the event on the launch took 2.5-2.8 us less
// each (8 MiB 7.5 -> 5.0 us, 32 MiB 15.0 -> 12.3 us), 0.5 us of them host time,
// and a wait for the event ended 2.4 us earlier.
hipError_t launch_swap(const SwapLaunch& a, hipStream_t stream, uint64_t* launches = nullptr,
                       hipEvent_t done = nullptr);

// Enqueues one HBM yardstick over `bytes` (a multiple of 16) of device
// memory with the swap kernels' copy loop: mode 0 copies src to dst, mode 1
// reads src only, mode 2 writes dst only (see aqua_hbm_yardstick).
hipError_t launch_yardstick(int mode, const uint8_t* src, uint8_t* dst, uint64_t bytes,
                            uint32_t key, hipStream_t stream);

// A range copy between two device-accessible addresses, in 64 KiB pieces.
struct CopyLaunch {
    const uint8_t* src;
    uint8_t* dst;
    const CopyDesc* descs;    // device-accessible, one per piece
    const InlineRanges* inl;  // if not null: the ranges, passed as a kernel argument instead
    uint32_t ranges;          // in *inl
    uint32_t pieces;
    uint32_t max_workgroups;  // 0: one workgroup per piece
};

// Enqueues it on `stream`; `done` as for launch_swap.
hipError_t launch_copy(const CopyLaunch& a, hipStream_t stream, hipEvent_t done = nullptr);

}  // namespace aqua
