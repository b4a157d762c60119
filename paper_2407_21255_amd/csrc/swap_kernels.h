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
    uint64_t min_run_bytes;
    uint64_t mean_run_bytes;  // per layer
    uint64_t max_run_bytes;
    uint32_t max_workgroups;  // 0: as many as part_grid says
    bool nt_pool_store;       // scatter: nontemporal stores into the pool
    bool xcd_units;           // a 1024-lane workgroup per unit instead of a wave per KiB,
                              // and to each XCD a contiguous eighth of the units
};

// Scatter store hint: nontemporal pool stores for chunks of 64 KiB and more, for
// calls of 2 GiB and more and for dealt calls of 256 MiB and more.  Measured on
// MI355X with a wave per KiB, nontemporal against ordinary stores: sorted and
// dealt swap-ins of an eighth of a 32-layer pool, three processes.
//   One call after another over 1 GiB of images and blocks in turn, so that the
//   caches hold nothing of the next: 64 KiB chunks 5-12 % shorter at every size
//   from 32 MiB to 3 GiB; 8 to 32 KiB chunks 8-12 % from 32 to 512 MiB, 10-15 %
//   at 1 and 3 GiB; 2 KiB chunks the same at 32 and 64 MiB, 9-11 % shorter from
//   128 MiB.  Each call waited for before the next: 0-5 % shorter up to 64 MiB,
//   4-11 % from 128 MiB.
//   The same call again and again on the same buffers, whose stores the 256 MB
//   last-level cache absorbs: 64 MiB 0-7 % longer, 128 to 256 MiB 4-16 %
//   longer (198 MiB of 16 KiB chunks 74.4 against 64.7 us; 64 KiB chunks 5-11 %),
//   512 MiB 5-12 % shorter.
//   Table order, 1 and 3 GiB: 4-8 % shorter.
// So the 256 MiB line is where ordinary stores end to win on cached buffers, and
// below it they lose on cold ones.  The 2 GiB line is older than the dealing:
// undealt calls of fewer bytes and smaller chunks keep ordinary stores, but
// only those of fewer than 16 blocks are left undealt there.
// The bytes are the whole call's for an HBM buffer, a slot's for the staged path.
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
// memory with the copy loop of whole-unit swaps and range copies: mode 0 copies src to dst, mode 1
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
