// swap_kernels.hip -- gfx950 gather (swap-out) and scatter (swap-in) kernels.
//
// The work is pure data movement (Aqua, section 7, "Efficient context
// switching"): no arithmetic on the values, so no MFMA and no LDS.  What bounds
// it is HBM, its write side above all, and for short runs the rate at which
// waves start.  A unit of work is one run of chunks in one layer; it is cut into
// parts of about 1 KiB, each copied by a workgroup of one wave with one 16-byte
// vector per lane, and the parts of a unit stay on one XCD (part_grid).
// Capped grids (zero-copy host swaps) and large calls in XCD unit order use
// 1024-lane workgroups that take whole units, kUnroll = 4 loads per lane in flight.
// The run descriptor is uniform across the workgroup and is fetched with
// scalar loads.  Cache hints: the offload side is written (swap-out) or read (swap-in) with
// nontemporal hints: it is touched once and should not displace the pool's
// working set in L2 and MALL.  The gather's pool loads are nontemporal too;
// the scatter's pool stores are nontemporal or ordinary by chunk size, bytes
// and run order (nt_pool_store).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "aqua_core.h"
#include "swap_kernels.h"

namespace aqua {

namespace {

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// Cache hints.  The defaults are the shipped configuration; the macros
// exist so that measurement sweeps can build variants.
#ifndef AQUA_NT_OUT_LD   // swap-out: pool loads
#define AQUA_NT_OUT_LD 1
#endif
#ifndef AQUA_NT_OUT_ST   // swap-out: image stores
#define AQUA_NT_OUT_ST 1
#endif
#ifndef AQUA_NT_IN_LD    // swap-in: image loads
#define AQUA_NT_IN_LD 1
#endif
// Swap-in pool stores: nontemporal or not is chosen per call
// (SwapLaunch::nt_pool_store).
#ifndef AQUA_YS_NT       // yardsticks: nontemporal loads and stores
#define AQUA_YS_NT 1
#endif

template <bool NT>
__device__ __forceinline__ v4u ld(const v4u* p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT>
__device__ __forceinline__ void st(v4u* p, v4u v) {
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Copies nvec 16-byte vectors from s to d with the whole workgroup of
// THREADS lanes: full passes of THREADS * kUnroll vectors, each lane's loads
// all issued before its first store, then one partial pass in which a lane
// copies only those of its kUnroll vectors that fall inside the span.  In the
// partial pass the gfx950 code waits for each conditional load before issuing
// the next; a form without lane branches that kept them all in flight
// measured no faster on 32 and 16 KiB chunks (within 1 %; one 32 KiB
// gather 2.5 % slower), and neither did workgroups that copy two 32 KiB
// units with all four loads of each lane in flight (1.5-8 % slower).
template <int THREADS, bool NT_LD, bool NT_ST>
__device__ __forceinline__ void copy_span(const v4u* __restrict__ s,
                                          v4u* __restrict__ d, uint32_t nvec) {
    const uint32_t t = threadIdx.x;
    constexpr uint32_t step = THREADS * kUnroll;
    uint32_t base = 0;
    for (; base + step <= nvec; base += step) {
        v4u r[kUnroll];
#pragma unroll
        for (int j = 0; j < (int)kUnroll; ++j) r[j] = ld<NT_LD>(s + base + j * THREADS + t);
#pragma unroll
        for (int j = 0; j < (int)kUnroll; ++j) st<NT_ST>(d + base + j * THREADS + t, r[j]);
    }
    if (base < nvec) {
        v4u r[kUnroll];
#pragma unroll
        for (int j = 0; j < (int)kUnroll; ++j) {
            const uint32_t i = base + j * THREADS + t;
            if (i < nvec) r[j] = ld<NT_LD>(s + i);
        }
#pragma unroll
        for (int j = 0; j < (int)kUnroll; ++j) {
            const uint32_t i = base + j * THREADS + t;
            if (i < nvec) st<NT_ST>(d + i, r[j]);
        }
    }
}

// OUT: pool -> image (gather).  !OUT: image -> pool (scatter), with
// nontemporal pool stores when NT_POOL_ST.
// Work unit u in [0, units) is (layer l0 + u / row, descriptor u % row), where
// row is ndesc or, with padding, layer_units(ndesc); layer l of the image side
// starts img_l0 layers before img_off's origin (0 for whole images, the first
// staged layer for a staging slot).  In plain order consecutive workgroups take consecutive units, whose runs the
// host may have dealt out to the XCDs (interleave_runs); with xcd_units each
// XCD takes a contiguous eighth of the units (xcd_unit).
// One unit: vectors [r.lo, r.lo + r.n) of run dsc in layer l.
template <bool OUT, bool NT_POOL_ST, int THREADS>
__device__ __forceinline__ void swap_unit(uint8_t* __restrict__ pool, uint8_t* __restrict__ img,
                                          const RunDesc& dsc, uint32_t l, uint32_t img_l0,
                                          VecRange r, uint64_t chunk_bytes,
                                          uint64_t pool_lstride) {
    uint8_t* p = pool + (uint64_t)l * pool_lstride + (uint64_t)dsc.block * chunk_bytes;
    uint8_t* m = img + dsc.img_off + (uint64_t)(l - img_l0) * dsc.img_lstride;
    if constexpr (OUT)
        copy_span<THREADS, AQUA_NT_OUT_LD, AQUA_NT_OUT_ST>(
            reinterpret_cast<const v4u*>(p) + r.lo, reinterpret_cast<v4u*>(m) + r.lo, r.n);
    else
        copy_span<THREADS, AQUA_NT_IN_LD, NT_POOL_ST>(
            reinterpret_cast<const v4u*>(m) + r.lo, reinterpret_cast<v4u*>(p) + r.lo, r.n);
}

__device__ __forceinline__ uint32_t run_vectors(const RunDesc& dsc, uint64_t chunk_bytes) {
    return (uint32_t)((uint64_t)dsc.nchunks * chunk_bytes / 16);
}

// Most uncapped launches: a wave per part of a unit (part_grid says why).  The loop
// ends after one pass unless the launch has more parts than a dispatch counts.
template <bool OUT, bool NT_POOL_ST, typename Get>
__device__ __forceinline__ void swap_parts(
    uint8_t* __restrict__ pool, uint8_t* __restrict__ img, const Get& get, uint32_t ndesc,
    uint32_t row, uint32_t l0, uint32_t img_l0, uint32_t units, uint32_t parts, uint32_t total,
    uint64_t chunk_bytes, uint64_t pool_lstride) {
    for (uint32_t b = blockIdx.x; b < total; b += gridDim.x) {
        const UnitPart q = part_at(b, units, parts);
        const uint32_t l = q.unit / row, k = q.unit - l * row;
        if (q.unit >= units || k >= ndesc) continue;
        const RunDesc dsc = get(k);
        const VecRange r = part_range(run_vectors(dsc, chunk_bytes), parts, q.part);
        swap_unit<OUT, NT_POOL_ST, kPartThreads>(pool, img, dsc, l0 + l, img_l0, r, chunk_bytes,
                                                 pool_lstride);
    }
}

// Whole units to 1024-lane workgroups: capped launches, which loop over them, and
// those in XCD unit order, one workgroup per unit.
template <bool OUT, bool NT_POOL_ST, typename Get>
__device__ __forceinline__ void swap_units(
    uint8_t* __restrict__ pool, uint8_t* __restrict__ img, const Get& get, uint32_t ndesc,
    uint32_t l0, uint32_t img_l0, uint32_t units, uint64_t chunk_bytes, uint64_t pool_lstride,
    uint32_t xcd_units) {
    const uint32_t u0 =
        (xcd_units && gridDim.x == units) ? xcd_unit(blockIdx.x, units) : blockIdx.x;
    for (uint32_t u = u0; u < units; u += gridDim.x) {
        const uint32_t l = u / ndesc;
        const RunDesc dsc = get(u - l * ndesc);
        swap_unit<OUT, NT_POOL_ST, kMaxThreads>(pool, img, dsc, l0 + l, img_l0,
                                                VecRange{0, run_vectors(dsc, chunk_bytes)},
                                                chunk_bytes, pool_lstride);
    }
}

// Each in two forms.  Runs in device-accessible memory (the pinned ring, the
// device ring or the scratch):
template <bool OUT, bool NT_POOL_ST>
__global__ __launch_bounds__(kPartThreads) void swap_runs_kernel(
    uint8_t* __restrict__ pool, uint8_t* __restrict__ img, const RunDesc* __restrict__ descs,
    uint32_t ndesc, uint32_t row, uint32_t l0, uint32_t img_l0, uint32_t units, uint32_t parts,
    uint32_t total, uint64_t chunk_bytes, uint64_t pool_lstride) {
    swap_parts<OUT, NT_POOL_ST>(
        pool, img, [&](uint32_t k) { return descs[k]; }, ndesc, row, l0, img_l0, units, parts,
        total, chunk_bytes, pool_lstride);
}

template <bool OUT, bool NT_POOL_ST>
__global__ __launch_bounds__(kMaxThreads) void swap_runs_whole_kernel(
    uint8_t* __restrict__ pool, uint8_t* __restrict__ img, const RunDesc* __restrict__ descs,
    uint32_t ndesc, uint32_t l0, uint32_t img_l0, uint32_t units, uint64_t chunk_bytes,
    uint64_t pool_lstride, uint32_t xcd_units) {
    swap_units<OUT, NT_POOL_ST>(
        pool, img, [&](uint32_t k) { return descs[k]; }, ndesc, l0, img_l0, units, chunk_bytes,
        pool_lstride, xcd_units);
}

// and runs in the kernel's arguments, for calls of at most kInlineRuns runs: a
// workgroup's descriptor comes from the argument segment instead of over the
// host link, and the call needs no ring space, no upload kernel and no device
// scratch.  A 32 MiB allocation-free round trip went from four launches and
// 42 us to two and 34 us.
template <bool OUT, bool NT_POOL_ST, uint32_t CAP>
__global__ __launch_bounds__(kPartThreads) void swap_runs_inline_kernel(
    uint8_t* __restrict__ pool, uint8_t* __restrict__ img, const InlineArg<CAP> runs,
    uint32_t ndesc, uint32_t row, uint32_t l0, uint32_t img_l0, uint32_t units, uint32_t parts,
    uint32_t total, uint64_t chunk_bytes, uint64_t pool_lstride) {
    swap_parts<OUT, NT_POOL_ST>(
        pool, img, [&](uint32_t k) { return unpack_inline(runs.run[k]); }, ndesc, row, l0, img_l0,
        units, parts, total, chunk_bytes, pool_lstride);
}

template <bool OUT, bool NT_POOL_ST>
__global__ __launch_bounds__(kMaxThreads) void swap_runs_inline_whole_kernel(
    uint8_t* __restrict__ pool, uint8_t* __restrict__ img, const InlineRuns runs, uint32_t ndesc,
    uint32_t l0, uint32_t img_l0, uint32_t units, uint64_t chunk_bytes, uint64_t pool_lstride,
    uint32_t xcd_units) {
    swap_units<OUT, NT_POOL_ST>(
        pool, img, [&](uint32_t k) { return unpack_inline(runs.run[k]); }, ndesc, l0, img_l0,
        units, chunk_bytes, pool_lstride, xcd_units);
}

// Range copy between two offload buffers (image migration): work unit u
// copies piece get(u).  With one workgroup per piece the XCDs take windows of
// adjacent pieces (xcd_window_unit); a capped grid loops in plain order.
template <typename Get>
__device__ __forceinline__ void copy_pieces(const uint8_t* __restrict__ src,
                                            uint8_t* __restrict__ dst, const Get& get,
                                            uint32_t n) {
    const uint32_t u0 = gridDim.x == n ? xcd_window_unit(blockIdx.x, n) : blockIdx.x;
    for (uint32_t u = u0; u < n; u += gridDim.x) {
        const CopyDesc dsc = get(u);
        copy_span<kMaxThreads, true, true>(reinterpret_cast<const v4u*>(src + dsc.src_off),
                                           reinterpret_cast<v4u*>(dst + dsc.dst_off),
                                           (uint32_t)(dsc.len / 16));
    }
}

__global__ __launch_bounds__(kMaxThreads) void copy_ranges_kernel(
    const uint8_t* __restrict__ src, uint8_t* __restrict__ dst,
    const CopyDesc* __restrict__ descs, uint32_t n) {
    copy_pieces(src, dst, [&](uint32_t u) { return descs[u]; }, n);
}

__global__ __launch_bounds__(kMaxThreads) void copy_ranges_inline_kernel(
    const uint8_t* __restrict__ src, uint8_t* __restrict__ dst, const InlineRanges ranges,
    uint32_t count, uint32_t n) {
    copy_pieces(src, dst, [&](uint32_t u) { return piece_of(ranges, count, u); }, n);
}

// HBM yardsticks over nvec contiguous vectors, in 64 KiB pieces with the lane
// shape and hints of whole-unit swap launches.  MODE 0 copies src to dst, MODE 1 only
// reads src (the vectors are folded together and stored to dst only if the
// fold equals a key no real input produces, so the loads stay), MODE 2 only
// writes dst: vector i holds {i low, i high, key, ~key}.
template <int MODE>
__global__ __launch_bounds__(kMaxThreads) void yardstick_kernel(
    const v4u* __restrict__ src, v4u* __restrict__ dst, uint64_t nvec, uint32_t key) {
    constexpr uint32_t per = kMaxThreads * kUnroll;
    const uint64_t units = (nvec + per - 1) / per;
    const uint32_t t = threadIdx.x;
    v4u acc = {0u, 0u, 0u, 0u};
    for (uint64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const uint64_t base = u * per;
        const uint32_t n = (uint32_t)std::min<uint64_t>(per, nvec - base);
        if constexpr (MODE == 0) {
            copy_span<kMaxThreads, AQUA_YS_NT, AQUA_YS_NT>(src + base, dst + base, n);
        } else if constexpr (MODE == 1) {
            v4u r[kUnroll];
#pragma unroll
            for (int j = 0; j < (int)kUnroll; ++j) {
                const uint32_t i = j * kMaxThreads + t;
                r[j] = i < n ? ld<AQUA_YS_NT>(src + base + i) : v4u{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int j = 0; j < (int)kUnroll; ++j) acc ^= r[j];
        } else {
#pragma unroll
            for (int j = 0; j < (int)kUnroll; ++j) {
                const uint32_t i = j * kMaxThreads + t;
                const uint64_t g = base + i;
                if (i < n)
                    st<AQUA_YS_NT>(dst + g, v4u{(uint32_t)g, (uint32_t)(g >> 32), key, ~key});
            }
        }
    }
    if constexpr (MODE == 1) {
        if (acc.x == key && acc.y == ~key && acc.z == key && acc.w == ~key) dst[0] = acc;
    }
}

// One launch; `done`, if given, completes with it (see launch_swap).
hipError_t launch_with_event(const void* fn, uint32_t grid, uint32_t threads, void** args,
                             hipStream_t stream, hipEvent_t done) {
    if (!done) return hipLaunchKernel(fn, dim3(grid), dim3(threads), args, 0, stream);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone)
        return hipExtLaunchKernel(fn, dim3(grid), dim3(threads), args, 0, stream, nullptr, done,
                                  0);
    (void)hipGetLastError();
    const hipError_t e = hipLaunchKernel(fn, dim3(grid), dim3(threads), args, 0, stream);
    return e == hipSuccess ? hipEventRecord(done, stream) : e;
}

template <bool OUT, bool NT_POOL_ST>
hipError_t launch_swap_k(const SwapLaunch& a, uint32_t l0, uint32_t nl, hipStream_t stream,
                         hipEvent_t done) {
    const bool whole = a.max_workgroups != 0 || a.xcd_units;
    const uint32_t row = whole ? a.ndesc : layer_units(a.ndesc);
    const uint32_t units = nl * row;
    const PartGrid g = part_grid(units, a.min_run_bytes, a.mean_run_bytes, a.max_run_bytes);
    const uint32_t grid = whole ? launch_grid(units, a.max_workgroups) : g.grid;
    const uint32_t threads = whole ? kMaxThreads : kPartThreads;
    // The argument array hands the runtime the runs where they are; passed by
    // value they would be copied once more.  The shorter argument is a prefix
    // of the longer one.
    const uint32_t xcd = a.xcd_units;
    const void* runs = a.inl ? (const void*)a.inl : (const void*)&a.descs;
    const void* part_args[] = {&a.pool, &a.img,   runs,     &a.ndesc, &row,           &l0,
                               &a.img_l0, &units, &g.parts, &g.total, &a.chunk_bytes,
                               &a.pool_lstride};
    const void* whole_args[] = {&a.pool,   &a.img, runs,           &a.ndesc,        &l0,
                                &a.img_l0, &units, &a.chunk_bytes, &a.pool_lstride, &xcd};
    const void* fn;
    if (!a.inl)
        fn = whole ? reinterpret_cast<const void*>(&swap_runs_whole_kernel<OUT, NT_POOL_ST>)
                    : reinterpret_cast<const void*>(&swap_runs_kernel<OUT, NT_POOL_ST>);
    else if (whole)
        fn = reinterpret_cast<const void*>(&swap_runs_inline_whole_kernel<OUT, NT_POOL_ST>);
    else if (a.ndesc <= kInlineFew)
        fn = reinterpret_cast<const void*>(&swap_runs_inline_kernel<OUT, NT_POOL_ST, kInlineFew>);
    else
        fn = reinterpret_cast<const void*>(&swap_runs_inline_kernel<OUT, NT_POOL_ST, kInlineRuns>);
    return launch_with_event(fn, grid, threads,
                             const_cast<void**>(whole ? whole_args : part_args), stream, done);
}

}  // namespace

hipError_t launch_copy(const CopyLaunch& a, hipStream_t stream, hipEvent_t done) {
    if (!a.pieces) return done ? hipEventRecord(done, stream) : hipSuccess;
    const uint32_t grid = launch_grid(a.pieces, a.max_workgroups);
    const void* inl[] = {&a.src, &a.dst, a.inl, &a.ranges, &a.pieces};
    const void* ring[] = {&a.src, &a.dst, &a.descs, &a.pieces};
    const void* fn = a.inl ? reinterpret_cast<const void*>(&copy_ranges_inline_kernel)
                           : reinterpret_cast<const void*>(&copy_ranges_kernel);
    return launch_with_event(fn, grid, kMaxThreads, const_cast<void**>(a.inl ? inl : ring), stream,
                             done);
}

hipError_t launch_swap(const SwapLaunch& a, hipStream_t stream, uint64_t* launches,
                       hipEvent_t done) {
    if (!a.ndesc || !a.num_layers) return done ? hipEventRecord(done, stream) : hipSuccess;
    // Whole layers per launch, fewer than 2^31 units each.
    const uint32_t per = layers_per_launch(layer_units(a.ndesc));
    const uint32_t end = a.first_layer + a.num_layers;
    for (uint32_t l0 = a.first_layer; l0 < end; l0 += per) {
        const uint32_t nl = std::min<uint32_t>(per, end - l0);
        const hipEvent_t last = l0 + nl == end ? done : nullptr;
        const hipError_t e = a.out ? launch_swap_k<true, false>(a, l0, nl, stream, last)
                             : a.nt_pool_store
                                 ? launch_swap_k<false, true>(a, l0, nl, stream, last)
                                 : launch_swap_k<false, false>(a, l0, nl, stream, last);
        if (e != hipSuccess) return e;
        if (launches) ++*launches;
    }
    return hipSuccess;
}

hipError_t launch_yardstick(int mode, const uint8_t* src, uint8_t* dst, uint64_t bytes,
                            uint32_t key, hipStream_t stream) {
    const uint64_t nvec = bytes / 16;
    if (!nvec) return hipSuccess;
    const uint64_t per = (uint64_t)kMaxThreads * kUnroll;
    const uint32_t grid = launch_grid((nvec + per - 1) / per, 0);
    const v4u* s = reinterpret_cast<const v4u*>(src);
    v4u* d = reinterpret_cast<v4u*>(dst);
    switch (mode) {
        case 0: hipLaunchKernelGGL(yardstick_kernel<0>, dim3(grid), dim3(kMaxThreads), 0, stream,
                                   s, d, nvec, key); break;
        case 1: hipLaunchKernelGGL(yardstick_kernel<1>, dim3(grid), dim3(kMaxThreads), 0, stream,
                                   s, d, nvec, key); break;
        case 2: hipLaunchKernelGGL(yardstick_kernel<2>, dim3(grid), dim3(kMaxThreads), 0, stream,
                                   s, d, nvec, key); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace aqua
