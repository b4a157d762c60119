// aqua_core.h -- host-side core of the KV page-swap library: argument
// validation, run planning, cross-stream hazard tracking and the swap
// space's range allocator.  Pure C++17,
// no HIP types, so that it builds and is tested on a machine without a GPU.
#pragma once

#include <cstddef>
#include <cstdint>
#include <map>
#include <unordered_map>
#include <utility>
#include <vector>

#include "aqua.h"

namespace aqua {

// Pool geometry.  One (layer, block) chunk of the pool
// [L][N][2][H][T][D] is C = 2*H*T*D*elem contiguous bytes.
struct Shape {
    uint32_t L = 0, N = 0, H = 0, T = 0, D = 0;
    int32_t dtype = 0;
    uint64_t C = 0;          // chunk bytes
    uint64_t pool_bytes = 0; // L*N*C
};

// Largest chunk (1 GiB) and largest pool or image (2^62 bytes) accepted.
constexpr uint64_t kMaxChunkBytes = 1ull << 30;
constexpr uint64_t kMaxBytes = 1ull << 62;

// Fills *out from a descriptor; AQUA_ERR_INVALID for a zero dimension, an
// unknown dtype, or a chunk that is not a multiple of 16 bytes.
aqua_status make_shape(const aqua_kv_desc* d, Shape* out);

// One swap call as the caller described it.
struct CallArgs {
    uint32_t num_seqs = 0;
    const int32_t* ids = nullptr;
    const uint64_t* offs = nullptr;        // num_seqs+1 CSR offsets
    const uint64_t* img_offsets = nullptr; // nullptr: packed images
    uintptr_t buf = 0;                     // offload buffer address
    uint64_t buf_bytes = 0;
    bool is_in = false;                    // swap-in: destinations are blocks
    // Blocks per layer of each image (>= its table length; the table covers
    // the first blocks of every layer).  nullptr: the table lengths.
    const uint64_t* img_blocks = nullptr;
    // Layers moved: [first_layer, first_layer + num_layers); 0 layers with
    // first_layer 0 means every layer.
    uint32_t first_layer = 0;
    uint32_t num_layers = 0;
};

// Blocks per layer of sequence k's image.
uint64_t image_blocks(const CallArgs& a, uint32_t k);

// One range of a migration: len bytes from src_off to dst_off.
struct CopyRange {
    uint64_t src_off, dst_off, len;
};

// Migration validation: offsets and lengths multiples of 16, ranges inside
// their buffers, destination ranges disjoint from each other and from every
// source range (as addresses).  Same codes and precedence as the oracle.
aqua_status validate_migrate(uintptr_t src, uint64_t src_bytes, uintptr_t dst,
                             uint64_t dst_bytes, uint32_t n, const uint64_t* src_off,
                             const uint64_t* dst_off, const uint64_t* len);

// Work item of the range-copy kernel: a piece of at most kCopyPiece bytes, or,
// in the kernel's arguments, a whole range and the index of its first piece.
constexpr uint64_t kCopyPiece = 64ull << 10;
struct alignas(16) CopyDesc {
    uint64_t src_off;
    uint64_t dst_off;
    uint64_t len;
    uint64_t first_piece;
};
static_assert(sizeof(CopyDesc) == 32, "descriptor layout is shared with the kernels");

// The ranges of a copy of few ranges, carried in the kernel's arguments; each
// workgroup finds its piece's range by bisection, six steps at most in the
// scalar cache.  Planning, writing and uploading one descriptor per piece took
// 88 us of host time and an 18 us kernel for 1.3 GiB in eight ranges; this takes
// neither.
constexpr uint32_t kInlineRanges = 64;
struct InlineRanges {
    CopyDesc range[kInlineRanges];
};
// Fills *out with the non-empty ranges and returns their pieces; *count is the
// number of ranges.  0 pieces with *count > kInlineRanges: too many to go there.
uint64_t pack_ranges(uint32_t n, const uint64_t* src_off, const uint64_t* dst_off,
                     const uint64_t* len, InlineRanges* out, uint32_t* count);
// Piece u of the packed ranges, u below their pieces.
constexpr CopyDesc piece_of(const InlineRanges& r, uint32_t count, uint64_t u) {
    uint32_t lo = 0, hi = count;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (r.range[mid].first_piece <= u)
            lo = mid;
        else
            hi = mid;
    }
    const CopyDesc& q = r.range[lo];
    const uint64_t at = (u - q.first_piece) * kCopyPiece, left = q.len - at;
    return CopyDesc{q.src_off + at, q.dst_off + at, left < kCopyPiece ? left : kCopyPiece, u};
}

// Splits the ranges into pieces of at most `unit` bytes.
size_t plan_copies(uint32_t n, const uint64_t* src_off, const uint64_t* dst_off,
                   const uint64_t* len, uint64_t unit, std::vector<CopyDesc>* out);

// One copy over the host link.
struct LinkPiece {
    void* dst;
    const void* src;
    uint64_t bytes;
};
// Appends a copy, as part of the last one where it continues that on both
// sides: a copy engine spends about 34 us on each copy beyond its bytes, so 36
// sequences of 1.2 MiB took 1.2 ms more than one copy of them all.
void append_piece(std::vector<LinkPiece>* v, const LinkPiece& p);

// Work item of the copy kernels: a run of `nchunks` consecutive pool blocks
// starting at `block` whose image chunks are also consecutive.  In layer l
// the pool side starts at (l*N + block)*C and the image side at
// img_off + l*img_lstride.  32 bytes so that one scalar load fetches it.
struct alignas(16) RunDesc {
    uint64_t img_off;
    uint64_t img_lstride;
    uint32_t block;
    uint32_t nchunks;
    uint32_t reserved0;
    uint32_t reserved1;
};
static_assert(sizeof(RunDesc) == 32, "descriptor layout is shared with the kernels");

// The runs of a small call, carried in the kernel's arguments: 16 bytes each,
// offsets in 16-byte vectors.  A kernel's argument segment holds 4 KiB, of
// which the other and the hidden arguments take about 350 bytes.  Measured on
// MI355X against reading the runs from the pinned ring, where a workgroup's
// first load crosses the host link: an 8 MiB swap's kernel 1.0 us of 5.8
// shorter, a 32 MiB one 1.1 us of 14; as fast as runs already in HBM, without
// the kernel that brings them there.
struct InlineRun {
    uint32_t block, nchunks, img_off16, img_lstride16;
};
constexpr uint32_t kInlineRuns = 224;
// A call of few runs takes a shorter argument: the host copies all of it.
constexpr uint32_t kInlineFew = 32;
template <uint32_t CAP>
struct InlineArg {
    InlineRun run[CAP];
};
using InlineRuns = InlineArg<kInlineRuns>;
// Fills *out from the runs; false (with *out unspecified) when there are more
// than kInlineRuns or an offset or stride is 64 GiB or more.
bool pack_inline(const std::vector<RunDesc>& runs, InlineRuns* out);
constexpr RunDesc unpack_inline(const InlineRun& r) {
    return RunDesc{(uint64_t)r.img_off16 * 16, (uint64_t)r.img_lstride16 * 16, r.block, r.nchunks,
                   0, 0};
}

// Where a call's `bytes` of descriptors go in a ring of `ring_bytes`: at the
// front when no live call's descriptors are there (the host then writes into
// lines it wrote a few calls ago, still in its caches; walking the whole ring
// wrote lines evicted long before, and copying a 135 KB plan into them took
// about 30 us), else at `head`, behind the last call's, or at the front again
// where that does not fit.  Never over a `kept` range: those are read again by
// graphs that captured a call.  False when the kept ranges leave no room.
using ByteRange = std::pair<uint64_t, uint64_t>;
bool ring_place(uint64_t ring_bytes, uint64_t bytes, uint64_t head,
                const std::vector<ByteRange>& live, const std::vector<ByteRange>& kept,
                uint64_t* lo);

// Launch geometry of the copy kernels.  A lane moves kUnroll 16-byte vectors
// per pass, its loads all issued before its first store, where a workgroup has
// as many for it: one of kMaxThreads lanes has 64 KiB in flight.
constexpr uint32_t kUnroll = 4;
constexpr uint32_t kMaxThreads = 1024;

// How an uncapped swap launch splits its units: each unit, one (layer, run), is
// cut into `parts` of about 1 KiB, each the work of a workgroup of one wave, one
// 16-byte vector per lane.  A wave ends, and its slot is refilled, as soon as
// its 1 KiB is stored; a 1024-lane workgroup holds the slots of its 16 waves
// until the last of its 64 KiB, and runs that are no multiple of 16 KiB leave
// some of them idle.  Measured on MI355X against one 1024-lane workgroup per unit
// (HBM traffic, 32 MiB to 5 GiB per call): 64 KiB chunks 5.95 -> 6.3 TB/s, 4 to
// 12 % at every size; 128 KiB 10 to 19 %; 32 KiB 1 to 10 %; 16 KiB 0 to 7 %; 8 KiB
// 4.9 -> 6.1 TB/s; 2 KiB 1.6 -> 5.5; one 1 MiB chunk in 32 layers 42 -> 14 us.  4 KiB
// parts of 256 lanes were as good from 512 MiB on, 8 KiB of 512 lanes 1-2 % behind,
// more vectors per lane 2-7 %.
// The parts of a unit go to the XCD the whole unit would go to (part_at), so
// that dealt runs stay dealt; below kSpreadUnits units they go to all XCDs.
constexpr uint32_t kXcdWays = 8;  // a launch's workgroups go to the 8 XCDs in turn
constexpr uint64_t kPartBytes = 1ull << 10;
constexpr uint32_t kPartThreads = 64;
constexpr uint32_t kSpreadUnits = 64;
// A dispatch counts its work-items in 32 bits: 2^25 workgroups of 64 lanes.
constexpr uint32_t kMaxPartGrid = 1u << 25;
struct PartGrid {
    uint32_t parts;  // per unit
    uint32_t total;  // indices for part_at: parts times the units, padded
    uint32_t grid;   // workgroups: total, at most kMaxPartGrid
};
// Runs of one length have as many parts as 1 KiB pieces.  Where lengths differ,
// the mean decides for large calls (workgroups past a short run's end return,
// and those of a long run copy more than 1 KiB) and the longest for small ones.
// A few longer runs among runs of one length do not count: one pair of adjacent
// blocks in a table lifts the mean above that length, and a part more is then a
// wave without work for every other run (2.5 GiB of 16 KiB chunks 1 % longer,
// 128 MiB of 1 KiB chunks with 16 pairs 87 against 57 us).  Where the shortest
// run is over eight ninths of the mean, it decides.
PartGrid part_grid(uint32_t units, uint64_t min_run_bytes, uint64_t mean_run_bytes,
                   uint64_t max_run_bytes);
// Units of one layer in such a launch, `ndesc` runs and padding: with a multiple
// of eight, run k goes to the same XCD in every layer.  Otherwise the XCDs take
// another eighth of the runs in each layer, and where the runs are read from the
// pinned ring each XCD fetches most of them over the link, all its waves
// waiting.  Measured on MI355X, runs of 8 to 96 KiB, 1 to 5 beyond a multiple
// of eight, padded against not: 4 layers 0-12 % shorter from 233 runs
// on (4091 runs of 64 KiB, 403 -> 360 us), 32 layers 0-3 %, 80 layers within
// 1 %; 1 GiB of 1 KiB runs in 32 layers 668 -> 464 us.  Runs in the kernel's
// arguments, at most kInlineRuns, only pay for the padding: 65 runs 1-7 % longer,
// 129 runs 0-4 %.
constexpr uint32_t kAlignRuns = 256;
constexpr uint32_t layer_units(uint32_t ndesc) {
    return ndesc < kAlignRuns ? ndesc : (ndesc + kXcdWays - 1) / kXcdWays * kXcdWays;
}
struct UnitPart {
    uint32_t unit, part;  // unit >= units: padding, nothing to do
};
// Index b of a launch's total: a bijection onto (unit, part), and padding.
constexpr UnitPart part_at(uint32_t b, uint32_t units, uint32_t parts) {
    if (units < kSpreadUnits) return UnitPart{b / parts, b % parts};
    const uint32_t j = b / 8;
    return UnitPart{j / parts * 8 + b % 8, j % parts};
}
// 16-byte vectors [lo, lo + n) of a run's nvec that part `part` copies.
struct VecRange {
    uint32_t lo, n;
};
constexpr VecRange part_range(uint32_t nvec, uint32_t parts, uint32_t part) {
    const uint32_t even = nvec / parts + (nvec % parts != 0);
    const uint32_t per = (even + kPartThreads - 1) / kPartThreads * kPartThreads;
    const uint64_t lo = (uint64_t)part * per;
    if (lo >= nvec) return VecRange{nvec, 0};
    return VecRange{(uint32_t)lo, nvec - (uint32_t)lo < per ? nvec - (uint32_t)lo : per};
}

// Workgroups of one launch over `units` work units: one per unit, at most
// `max_workgroups` when that is non-zero, and never more than kMaxGrid.  A
// dispatch counts its work-items in 32 bits, so 1024-lane workgroups allow
// at most 4 194 303 of them; the kernels loop over units with a grid
// stride, so a capped grid still covers every unit.
constexpr uint32_t kMaxGrid = 1u << 21;
uint32_t launch_grid(uint64_t units, uint32_t max_workgroups);

// The order in which a call's runs go to the kernels (each run is
// independent, so the order changes no byte).  Runs dealt out to the XCDs
// (interleave_runs), swap-ins sorted by pool block first:
//   chunks of 64 KiB or more: every swap-in; a swap-out when it covers at
//     least 40 % of the pool's blocks or its sequences average at least 32
//     blocks (the others keep table order);
//   smaller chunks: a swap-in that covers at least 40 % of the pool; every
//     other call keeps table order.
// Sorted, the pool side of consecutive units moves through the pool in
// address order and the image side jumps; in table order the reverse.
// Measured on MI355X, same box, with one 1024-lane workgroup per unit:
//   swap-ins (pool written in order), calls covering half the pool: sorted
//     against table order, 70B scatter 3.3 % shorter, one TP2 rank's 1.6 %,
//     one TP4 rank's 2.8 %; a sixteenth of the pool (8B, fp8 8B): no gain,
//     a quarter (the preemption cycle): 3-7 % longer;
//   swap-outs (image written in order in table order), half the pool: sorted
//     against table order, 64 KiB chunks 4.5 % shorter but 32 KiB chunks
//     1.6 % and 16 KiB chunks 6 % longer; once dealt to the XCDs, the 70B
//     gather in table order took 2.8 % less than sorted (3.53 against
//     3.63 ms, four runs each), the pair +1.4 %.
//   sparse calls of 64 KiB chunks, dealt as above against table order
//     (three runs each): one prompt of 1024 or 2048 blocks +3 to +7.5 %,
//     8 prompts +1.3 to +2.7 %, the 8B pair +1.1 %, prefix loads beside
//     other swaps +3.6 %, 64 prompts of 32 blocks +3 to +4 %; dealing the
//     gather of 64 prompts of 16 blocks too cost it 8 %, hence the 32-block
//     mean.  Sorting or dealing sparse calls of smaller chunks lost 2.6 %
//     (the fp8 8B pair, whose scatter then leaves the XCD unit order).
// With a wave per KiB the orders lie closer (64 KiB chunks, 32 layers, three
// processes): swap-outs dealt against table order 1 % longer to 4 % shorter at
// 128 MiB to 3 GiB, 32 sequences of 16 blocks 1 % shorter and no longer slower;
// swap-ins sorted and dealt against dealt alone within 1 %, against table order
// within 1 % at 256 MiB, 1-2 % shorter at 1 GiB, 0-2 % at 3 GiB.
enum class RunOrder { kTable, kSortedDealt, kTableDealt };
constexpr uint64_t kDenseMinPermille = 400;     // share of the pool's blocks
constexpr uint64_t kDealMinChunk = 64ull << 10;
constexpr uint64_t kDealOutMinMeanBlocks = 32;  // sparse swap-outs: blocks per sequence
RunOrder run_order(bool is_in, uint64_t chunk_bytes, uint64_t blocks, uint32_t num_blocks,
                   uint32_t num_seqs);

// run_order refined by the bytes a call of chunks under 64 KiB moves, for the
// calls that run_order leaves in table order.  Measured on MI355X with a wave
// per KiB, 32 layers, one and 16 sequences, a third to a twentieth of the pool,
// calls one after another on cold buffers, three processes:
//   swap-outs, dealt in table order: 128 MiB to 2.2 GiB within 2.5 % of table
//     order for chunks to 16 KiB, 3 % shorter to 1 % longer for 32 KiB; against
//     whole units in XCD unit order (32 KiB chunks) 3-9 % shorter at 128 MiB,
//     1-5 % at 512 MiB, 1-3 % at 1 GiB, within 1 % at 2.2 GiB;
//   swap-ins, dealt against table order: 2 KiB chunks 1 % shorter to 3 % longer,
//     8 KiB within 2 %, 16 KiB 0-4 % and 32 KiB 1-5 % shorter; against whole
//     units in XCD unit order (32 KiB) 0-9 % shorter up to 1 GiB;
//   swap-ins, sorted as well, against dealt alone: 1-4 % longer at 128 MiB; from
//     512 MiB on 8 to 32 KiB chunks 2-7 % shorter for a third and a twelfth of
//     the pool, 4 % shorter to 3 % longer for a twentieth; 2 KiB chunks 0-5 %
//     longer, for a twentieth 34-92 % (the sort, O(runs + pool blocks), then
//     outlasts the copy).  On another box, 4 to 80 layers, sorted within 3 % of
//     dealt alone from 256 MiB on where a block has 256 KiB over all layers, 2-5 %
//     longer below 256 MiB; where a block has 128 KiB 1 % shorter to 5 % longer,
//     and with 32 KiB (8 KiB chunks in 4 layers) up to 13 % longer, 64 MiB 81
//     against 31 us.  A call waited for takes the sort's time longer.  So only
//     calls that cover a sixteenth of the pool sort, of 256 MiB and more, with
//     256 KiB and more to a block.
//
// Calls of 2 GiB and more in chunks between 16 and 64 KiB, swap-outs and those
// swap-ins that cover less than 40 % of the pool, keep table order, and the
// kernels take whole units of them in XCD unit order (xcd_unit).  The line is drawn for a scheduler's slices, a
// swap-out beside a swap-in on two streams: the fp8 preemption cycle (32 KiB
// chunks, 2.05 GiB each way, sequences of very different lengths) took 1584 us
// with a wave per KiB in that order, 1583 dealt, 1509 so.  Lone calls and even
// slices, three processes, whole units in XCD unit order against
//                              24 KiB         32 KiB         48 KiB chunks
//   a wave per KiB in that order
//     swap-out, 2.1-5 GiB      2-3 % shorter  3-4 % shorter  0-1 % shorter
//     swap-in                  -3 to +3 %     within 1 %     3 % longer
//     both at once             0-4 % shorter  2-4 % shorter  1 % longer
//   dealt (swap-outs and swap-ins), a wave per KiB
//     swap-out                 within 2 %     -2 to +1 %     1-3 % longer
//     swap-in, 2.1-3 GiB       4-6 % longer   1-3 % longer   5-6 % longer
//     both at once             -4 to +2 %     0-2 % shorter  2-3 % longer
//   sorted and dealt swap-ins
//     swap-in, 2.1-3 GiB       3-6 % longer   8-10 % longer  4-6 % longer
//     both at once             3-7 % shorter  1-6 % shorter  1-2 % shorter
// (In one of the three processes 24 KiB swap-ins of 3 GiB in XCD unit order were
// 11 % shorter than dealt, in all three those of 5 GiB of an eighth of the pool.)
// A lone swap-in of that size would gain from being sorted and dealt, by which a
// slice would lose; the rule does not tell them apart.  Below 2 GiB lone calls
// are as short dealt or shorter, and slices of 24 and 48 KiB chunks 1-3 % shorter;
// those of 32 KiB chunks are 1-3 % longer (1.9 GiB 1340 against 1305 us).
// The bytes are the whole call's.
constexpr uint64_t kXcdUnitMinBytes = 2ull << 30;
constexpr uint64_t kSortMinShare = 16;  // a sixteenth of the pool's blocks
constexpr uint64_t kSortMinBytes = 256ull << 20;
constexpr uint64_t kSortMinRow = 256ull << 10;  // a block's bytes over the call's layers
RunOrder call_order(bool is_in, uint64_t chunk_bytes, uint64_t blocks, uint32_t num_blocks,
                    uint32_t num_seqs, uint64_t call_bytes);

// Puts the runs in ascending order of their first block, keeping the table
// order of runs that start at the same block (a swap-out may name a block
// twice).  A counting sort over the pool's blocks, O(runs + num_blocks), when
// the runs number at least a sixteenth of the blocks; a stable comparison
// sort, O(runs log runs), below that, so that a small call does not pay for
// the whole pool.  `counts` and `tmp` are reusable scratch.
constexpr uint64_t kSortCountingMinRatio = 16;
void sort_by_block(std::vector<RunDesc>* runs, uint32_t num_blocks,
                   std::vector<uint32_t>* counts, std::vector<RunDesc>* tmp);

// XCD-aware order of a dense call's runs.  A launch's workgroups go to
// MI355X's 8 XCDs (each with its own L2) in turn, and the kernels take one
// unit per workgroup, layer by layer.  Dealing a layer's runs out 8 ways (run
// j of the result is run j / 8 of the (j % 8)-th contiguous eighth of the
// input; the first n % 8 eighths hold one run more) gives each XCD one
// contiguous eighth of the runs in every layer:
// of the pool range when they are sorted, of the image when they are in
// table order, instead of every XCD taking every eighth run of one shared
// range.  Measured on MI355X against sorted order, same box, 3 to 6 runs
// each: 70B pair +1.4 to +3.3 % (four comparisons), one TP4 rank +2.7 to
// +3.3 %, the Yi-34B prefix load +2.1 to +3.6 %, one TP2 rank +1.0 %; the
// fair-scheduling reschedules -0.4 to -1.7 % (within their run-to-run
// spread).  2 ways gained about half as much, 16 or 32 ways lost 1-4 %
// against 8.  Which calls are dealt is run_order's rule.  A launch may start
// its turn at another XCD than the first (where the previous launch left
// off); that only changes which XCD takes which eighth.  Runs only ever
// change order, so no byte changes.  `tmp` is reusable scratch.
void interleave_runs(std::vector<RunDesc>* runs, uint32_t ways, std::vector<RunDesc>* tmp);

// XCD-aware unit order inside the kernels, on a launch of one workgroup per
// unit: workgroup b (sent to XCD (b + c) % 8, c fixed for the launch) takes unit
// xcd_unit(b, units), so that each XCD copies one contiguous eighth of the
// launch's units in order (the (b % 8)-th eighth; the first units % 8 eighths
// hold one unit more).  A bijection on [0, units).  For undealt calls of 2 GiB
// and more, chunks between 16 and 64 KiB (exclusive), to an HBM buffer; call_order
// says what it measures there.  When every undealt call was of one 1024-lane
// workgroup per unit, it cost 64 KiB chunks 6 % (64 short prompts) and 16 KiB
// chunks 1.2 % (a TP4 rank), so those never take it.
constexpr uint32_t xcd_unit(uint32_t block, uint32_t units) {
    const uint32_t x = block % kXcdWays, q = units / kXcdWays, r = units % kXcdWays;
    return x * q + (x < r ? x : r) + block / kXcdWays;
}
// The same within windows of 64 units, for a copy of contiguous pieces: each
// XCD takes eight adjacent 64 KiB pieces of a 4 MiB window.  A bijection on
// [0, units).  Measured on MI355X against plain order: 1.3 GiB 495 -> 438 us,
// 4 GiB 1637 -> 1390 us (5.25 -> 6.18 TB/s), 256 MiB 90 -> 87 us, 64 MiB and
// less the same.  Windows of 8 to 32 units gained half as much at most; one
// window over the whole copy as much at 1 GiB, but 64 MiB took 25 % longer.
constexpr uint32_t kXcdWindow = 64;
constexpr uint32_t xcd_window_unit(uint32_t block, uint32_t units) {
    const uint32_t base = block / kXcdWindow * kXcdWindow;
    return base + xcd_unit(block - base, units - base < kXcdWindow ? units - base : kXcdWindow);
}
constexpr uint64_t kXcdUnitMinChunk = 16ull << 10;  // exclusive
constexpr uint64_t kXcdUnitMaxChunk = 64ull << 10;  // exclusive
bool xcd_unit_order(uint64_t chunk_bytes, bool dealt);

// Layers per launch of a call with `ndesc` runs per layer: whole layers and
// fewer than 2^31 units per launch, so that almost every call is one launch.
// Launches of at most 512 MiB had made calls of 32 KiB chunks 3-5 % shorter
// in plain unit order; with the XCD unit order, which gives each XCD an
// eighth of a whole launch, one launch per call measured faster again (one
// TP2 rank +2.4 %, the fp8 preemption cycle and 8B pair +0.4 %, four runs
// each), and splitting 16 or 64 KiB calls lost 2-4 %.
uint32_t layers_per_launch(uint32_t ndesc);

// Reusable scratch for duplicate detection (epoch-stamped marks, O(n)).
struct DupMarks {
    std::vector<uint32_t> mark;
    uint32_t epoch = 0;
};

// Validation in the library's precedence: invalid -> range -> duplicate ->
// capacity.  Pointer classes are checked by the caller (they need HIP).
aqua_status validate_call(const Shape& s, const CallArgs& a, DupMarks& marks);

// Byte offset of sequence k's image inside the buffer.
uint64_t image_offset(const Shape& s, const CallArgs& a, uint32_t k);

// Coalesces each table into runs bt[i+1] == bt[i] + 1, split so that a run
// covers at most max(1, max_unit_bytes / C) chunks.  Appends to *out and
// returns the number of descriptors appended.
size_t plan_runs(const Shape& s, const CallArgs& a, uint64_t max_unit_bytes,
                 std::vector<RunDesc>* out);

// Half-open byte ranges [lo, hi) of the buffer that the call touches (one
// per non-empty sequence).
void image_ranges(const Shape& s, const CallArgs& a,
                  std::vector<std::pair<uint64_t, uint64_t>>* out);

// ---------------------------------------------------------------------------
// Hazard tracker.
//
// Every call gets a ticket (1, 2, 3, ...) and runs on a "lane" (one lane
// per distinct stream).  Work on one lane completes in issue order, so a
// dependency on ticket t of lane m is satisfied by waiting on the newest
// conflicting ticket of m.  Per pool block the tracker keeps the last
// writing ticket and, per lane, the newest ticket reading it since that
// write; per offload byte range it keeps the in-flight readers and writers.
// Tickets known complete (per-lane watermark) are never waited on.
//
// Memory stays bounded however many calls are issued: the lane of a ticket
// is kept only from the oldest ticket not yet known complete onwards (every
// older ticket is complete, whatever its lane), and a lane whose tickets
// have all completed can be handed to another stream (LaneMap).
class HazardTracker {
public:
    struct Dep {
        uint32_t lane;
        uint64_t ticket;
    };

    explicit HazardTracker(uint32_t num_blocks = 0) { reset(num_blocks); }
    void reset(uint32_t num_blocks);

    // What one call touches: pool blocks it reads or writes, and byte
    // ranges [lo, hi) of offload buffers (by address) it reads or writes.
    struct Access {
        const int32_t* blocks_read = nullptr;
        size_t n_blocks_read = 0;
        const int32_t* blocks_written = nullptr;
        size_t n_blocks_written = 0;
        const std::pair<uint64_t, uint64_t>* ranges_read = nullptr;
        size_t n_ranges_read = 0;
        const std::pair<uint64_t, uint64_t>* ranges_written = nullptr;
        size_t n_ranges_written = 0;
    };

    // Registers call `ticket` (must exceed every earlier ticket) on `lane`.
    // Writes into *deps, per other lane, the newest earlier ticket the call
    // must wait for.  Returns the number of conflicts that were skipped
    // because already complete.  Blocks written by one call must be
    // distinct; a range both read and written is listed as written.
    uint64_t issue(uint64_t ticket, uint32_t lane, const Access& a,
                   std::vector<Dep>* deps);

    // Everything on `lane` up to and including `ticket` has completed.
    void complete(uint32_t lane, uint64_t ticket);
    uint64_t completed(uint32_t lane) const;
    // Lane of an issued ticket that is not yet known complete; kNoLane for a
    // ticket already known complete (or never issued).
    static constexpr uint32_t kNoLane = UINT32_MAX;
    uint32_t lane_of(uint64_t ticket) const;
    // Known complete: below the oldest outstanding ticket, or at or below
    // its lane's watermark.
    bool done(uint64_t ticket) const;
    // Every ticket issued on `lane` is known complete.
    bool idle(uint32_t lane) const;
    size_t live_ranges() const { return ranges_.size(); }
    uint64_t last_ticket() const { return last_ticket_; }
    // Tickets whose lane is still kept (from the oldest one not known
    // complete to the newest) and lanes known to the tracker.
    size_t tickets_kept() const { return ticket_lane_.size() - head_; }
    size_t lanes() const { return done_.size(); }

private:
    struct Reader {
        uint32_t lane;
        uint64_t ticket;
    };
    // One pool block: its last writer and its readers since then, at most
    // one per lane.  The first reader is kept in the record, so that a call
    // touches one 24-byte record per block; readers on further lanes at
    // once (several streams reading one block) go to more_.
    struct BlockRec {
        uint64_t writer = 0;       // ticket of the last writer, 0: none
        uint64_t reader = 0;       // ticket of the kept reader, 0: none
        uint32_t reader_lane = 0;
        uint32_t more = 0;         // 1: more_ holds further readers of the block
    };
    struct RangeRec {
        uint64_t lo, hi, ticket;
        uint32_t lane;
        bool write;
    };
    // What issue() found for one earlier ticket (see need()).
    enum class Need : uint8_t { kNone, kComplete, kSameLane, kWait };
    void ensure_lane(uint32_t lane);
    void prune();
    Need need(uint64_t ticket, uint32_t lane);

    std::vector<BlockRec> blocks_;
    std::unordered_map<uint32_t, std::vector<Reader>> more_;
    std::vector<RangeRec> ranges_;
    std::vector<uint64_t> done_;         // per lane watermark
    std::vector<uint64_t> last_;         // per lane, newest ticket issued on it
    std::vector<uint64_t> dep_;          // per lane, scratch of one issue()
    std::vector<uint32_t> ticket_lane_;  // from head_: lanes of tickets base_, base_ + 1, ...
    size_t head_ = 0;
    uint64_t base_ = 1;                  // every ticket below is complete
    uint64_t last_ticket_ = 0;
};

// Stream -> lane map of one pool.  A stream seen before keeps its lane; a
// new stream takes over the lowest lane that is idle in the tracker (every
// ticket issued on it complete), else a new lane, so the lane count is at
// most the number of streams with calls in flight at once, plus one.
class LaneMap {
public:
    uint32_t lane_for(uintptr_t stream, const HazardTracker& t);
    size_t size() const { return stream_.size(); }
    uintptr_t stream_of(uint32_t lane) const { return stream_[lane]; }

private:
    std::vector<uintptr_t> stream_;
};

// First-fit allocator of byte ranges inside one arena [0, size) (the swap
// space's device region and its host region).  Every range starts on an
// `align` boundary and is a multiple of it; freeing coalesces neighbours.
// Host bookkeeping only: whoever reuses a freed range orders the reuse.
// Copy engines for the two link directions from the runtime's masks (bit e:
// engine e).  Per direction the candidates are the runtime's preferred
// engines that are available; else the `fast` engines (those that carry the
// host link at its rate) that are available; else the `fast` engines, shared
// with their other users, rather than a slower free one.  The lowest-numbered
// candidate is taken, the host-to-device direction on a different engine from
// the device-to-host one where its candidates allow.  With `fast` empty the
// available engines stand in for it.  -1 for a direction with no candidate.
void pick_link_engines(uint32_t d2h_avail, uint32_t d2h_pref, uint32_t h2d_avail,
                       uint32_t h2d_pref, uint32_t fast, int32_t* d2h, int32_t* h2d);

class RangeAllocator {
public:
    void reset(uint64_t size, uint64_t align);
    bool alloc(uint64_t bytes, uint64_t* off);  // false: no free range fits
    bool free(uint64_t off);                     // false: off is not allocated
    uint64_t size() const { return size_; }
    uint64_t free_bytes() const { return free_total_; }
    uint64_t largest_free() const;
    uint64_t granted(uint64_t off) const;        // bytes of the range at off (0: none)

private:
    uint64_t size_ = 0, align_ = 1, free_total_ = 0;
    std::map<uint64_t, uint64_t> free_;   // offset -> length
    std::map<uint64_t, uint64_t> used_;   // offset -> length
};

}  // namespace aqua
