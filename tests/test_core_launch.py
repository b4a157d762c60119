"""How a call's launches are shaped, host core alone (no GPU)."""
import ctypes
import os

import numpy as np
import pytest

from paper_2407_21255_amd import build
from tests import core_lib

K = 1 << 10


@pytest.mark.parametrize("ndesc", [1, 7, 63, 64, 224, 225, 255, 256, 257, 263, 264, 2047, 4091])
def test_runs_keep_their_xcd_from_layer_to_layer(ndesc):
    """Every run of every layer once; from 256 runs on, padded to a multiple of
    eight, each run on one XCD over all layers."""
    fn = core_lib.lib().aqua_core_layer_hits
    fn.argtypes, fn.restype = [ctypes.c_uint32] * 2 + [ctypes.c_void_p], ctypes.c_int32
    hits = np.zeros(5 * ndesc, dtype=np.uint8)
    same = fn(5, ndesc, hits.ctypes.data)
    assert (hits == 1).all()
    assert same == (ndesc % 8 == 0 or ndesc >= 256)


def _part_grid(units, mean, longest):
    fn = core_lib.lib().aqua_core_part_grid
    fn.argtypes = [ctypes.c_uint32, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_void_p]
    fn.restype = None
    out = np.zeros(3, dtype=np.uint32)
    fn(units, mean, longest, out.ctypes.data)
    return tuple(int(x) for x in out)     # parts, total, grid


@pytest.mark.parametrize("units,mean,longest,want", [
    (1, 16, 16, (1, 1, 1)), (63, 1024, 1024, (1, 63, 63)), (64, 1024, 1024, (1, 64, 64)),
    (65, 1025, 1025, (2, 144, 144)), (128, 64 * K, 64 * K, (64, 8192, 8192)),
    (163840, 64 * K, 64 * K, (64, 10485760, 10485760)),
    # Runs of several lengths: the longest decides for few waves, the mean for many.
    (8, 3 * K, 64 * K, (64, 512, 512)), (32768, 3 * K, 64 * K, (3, 98304, 98304)),
    # More parts than a dispatch counts: fewer, then a loop.
    (1 << 20, 64 * K, 64 * K, (32, 1 << 25, 1 << 25)),
    (1 << 25, 2 * K, 2 * K, (1, 1 << 25, 1 << 25)),
    ((1 << 31) - 1, 32, 32, (1, 1 << 31, 1 << 25)), (4, 1 << 30, 1 << 30, (1 << 20, 1 << 22, 1 << 22))])
def test_a_wave_per_kib_of_a_run(units, mean, longest, want):
    parts, total, grid = got = _part_grid(units, mean, longest)
    assert got == want
    assert grid * 64 < 1 << 32 and total >= units and total % parts == 0


@pytest.mark.parametrize("units,shortest,mean,longest,parts", [
    # One pair of adjacent blocks among 2047 runs of a block; 16 pairs among 4096.
    (163760, 16 * K, 16 * K + 8, 32 * K, 16), (130560, K, K + 4, 2 * K, 1),
    (65535, 1280, 1281, 2560, 2), (65535, 64 * K, 64 * K, 64 * K, 64),
    # Up to an eighth more than the shortest, and from there on, the mean.
    (65536, 8 * K, 9 * K - 16, 64 * K, 8), (65536, 8 * K, 9 * K, 64 * K, 9),
    # Most runs long, some short: the mean as before; few waves: the longest.
    (65536, 8 * K, 63 * K + 16, 64 * K, 64), (100, 16 * K, 16 * K + 8, 32 * K, 32)])
def test_few_longer_runs_give_the_others_no_empty_part(units, shortest, mean, longest, parts):
    fn = core_lib.lib().aqua_core_parts
    fn.argtypes = [ctypes.c_uint32] + [ctypes.c_uint64] * 3
    fn.restype = ctypes.c_uint32
    assert fn(units, shortest, mean, longest) == parts


@pytest.mark.parametrize("units", [1, 2, 7, 63, 64, 65, 71, 72, 130])
@pytest.mark.parametrize("lengths", [(1,), (64,), (65,), (4096,), (1, 64, 65, 700, 4096), (640, 641)])
def test_parts_cover_every_vector_once(units, lengths):
    """Over the whole index range of a launch every vector of every unit is
    copied exactly once, for one run length and for several, with as many
    parts as the rule gives, fewer and more."""
    fn = core_lib.lib().aqua_core_part_hits
    P = ctypes.c_void_p
    fn.argtypes, fn.restype = [ctypes.c_uint32] * 4 + [P, P, P], None
    nvec = np.array(lengths, dtype=np.uint32)
    n = len(nvec)
    per_unit = nvec[np.arange(units) % n].astype(np.uint64)
    base = np.concatenate([[0], np.cumsum(per_unit)]).astype(np.uint64)
    parts0, _, _ = _part_grid(units, int(nvec.mean() * 16), int(nvec.max()) * 16)
    slots = units if units < 64 else -(-units // 8) * 8
    for parts in sorted({1, 2, 3, parts0, parts0 + 1}):
        hits = np.zeros(int(base[-1]), dtype=np.uint8)
        fn(slots * parts, units, parts, n, nvec.ctypes.data, base.ctypes.data, hits.ctypes.data)
        assert (hits == 1).all(), parts


@pytest.mark.parametrize("units,lengths", [(1, (300,)), (63, (1, 64, 65)), (64, (130,)),
                                           (130, (1, 64, 65, 700)), (1000, (1,))])
def test_a_grid_smaller_than_the_launch_covers_it(units, lengths):
    """Workgroups that take index after index a grid apart (launches of more
    parts than a dispatch counts) copy every vector once, whatever the grid."""
    fn = core_lib.lib().aqua_core_grid_hits
    P = ctypes.c_void_p
    fn.argtypes, fn.restype = [ctypes.c_uint32] * 5 + [P, P, P], None
    nvec = np.array(lengths, dtype=np.uint32)
    per_unit = nvec[np.arange(units) % len(nvec)].astype(np.uint64)
    base = np.concatenate([[0], np.cumsum(per_unit)]).astype(np.uint64)
    parts, total, _ = _part_grid(units, int(nvec.mean() * 16), int(nvec.max()) * 16)
    for grid in sorted({1, 7, 8, 64, max(1, total // 2), max(1, total - 1), total}):
        hits = np.zeros(int(base[-1]), dtype=np.uint8)
        fn(grid, total, units, parts, len(nvec), nvec.ctypes.data, base.ctypes.data,
           hits.ctypes.data)
        assert (hits == 1).all(), grid


@pytest.mark.parametrize("units,mean,longest", [
    ((1 << 31) - 1, 32, 32), ((1 << 31) - 1, 64 * K, 64 * K), (1 << 25, 2 * K, 2 * K),
    ((1 << 25) + 1, 16, 16), (430000 * 80, 16, 16), (1 << 20, 64 * K, 1 << 30)])
def test_the_last_step_of_a_looping_grid_does_not_wrap(units, mean, longest):
    """An index and one grid more stay below 2^32, in which they are counted."""
    _, total, grid = _part_grid(units, mean, longest)
    assert total >= units and total - 1 + grid < 1 << 32


@pytest.mark.parametrize("chunk", [16, 8 * K, 16 * K, 16 * K + 16, 32 * K, 64 * K - 16, 64 * K])
def test_small_chunk_calls_are_dealt(chunk):
    """Chunks under 64 KiB: swap-outs dealt, swap-ins dealt and, from a
    sixteenth of the pool up, sorted; but 2 GiB and more in chunks between 16
    and 64 KiB (swap-ins: of a small part of the pool) stays in table order,
    which those kernels take in XCD unit order.  64 KiB follows run_order."""
    T, S, D = core_lib.TABLE, core_lib.SORTED_DEALT, core_lib.TABLE_DEALT
    G = 1 << 30
    if chunk == 64 * K:
        for is_in in (0, 1):
            for blocks, n, seqs in ((15, 4096, 1), (512, 4096, 64), (2048, 4096, 1)):
                assert core_lib.call_order(is_in, chunk, blocks, n, seqs, 4 * G) == \
                    core_lib.run_order(is_in, chunk, blocks, n, seqs)
        return
    between = 16 * K < chunk
    for seqs in (1, 64):
        assert core_lib.call_order(0, chunk, 15, 4096, seqs, G) == T
        assert core_lib.call_order(0, chunk, 16, 4096, seqs, G) == D
        assert core_lib.call_order(0, chunk, 2048, 4096, seqs, 2 * G - 1) == D
        assert core_lib.call_order(0, chunk, 2048, 4096, seqs, 2 * G) == (T if between else D)
        assert core_lib.call_order(1, chunk, 15, 4096, seqs, G) == T
        assert core_lib.call_order(1, chunk, 255, 4096, seqs, G) == D
        assert core_lib.call_order(1, chunk, 256, 4096, seqs, G) == S
        assert core_lib.call_order(1, chunk, 256, 4096, seqs, 2 * G - 1) == S
        assert core_lib.call_order(1, chunk, 256, 4096, seqs, 2 * G) == (T if between else S)
        assert core_lib.call_order(1, chunk, 2048, 4096, seqs, 4 * G) == S
    assert core_lib.call_order(1, chunk, 0, 0, 0, 0) == T


@pytest.mark.parametrize("layers,chunk,blocks,num_blocks,sorts", [
    (4, 8 * K, 2828, 36898, False),      # 88 MiB: the sort outlasts the copy
    (4, 8 * K, 32768, 131072, False),    # 1 GiB of 32 KiB blocks
    (16, 8 * K, 8192, 65536, False),     # 1 GiB of 128 KiB blocks
    (32, 8 * K, 1023, 8192, False), (32, 8 * K, 1024, 8192, True),     # 256 MiB, 256 KiB
    (31, 8 * K, 2048, 8192, False), (32, 8 * K, 1024, 16384, True), (32, 8 * K, 1024, 16385, False),
    (4, 8 * K, 32768, 65536, True), (4, 8 * K, 26214, 65536, False)])  # 40 %: run_order's rule
def test_only_calls_that_gain_by_it_are_sorted(layers, chunk, blocks, num_blocks, sorts):
    """Swap-ins of small chunks that cover less than 40 % of the pool: sorted
    from a sixteenth of it, 256 MiB and 256 KiB to a block, else dealt."""
    got = core_lib.call_order(1, chunk, blocks, num_blocks, 1, layers * blocks * chunk)
    assert got == (core_lib.SORTED_DEALT if sorts else core_lib.TABLE_DEALT)


@pytest.mark.parametrize("n", [0, 1, 223, 224, 225])
def test_runs_in_kernel_arguments_keep_every_field(n):
    """What a kernel reads from its arguments is the run that was planned, at
    the largest values that fit; one more run, or an offset or stride of
    64 GiB, goes by the ring instead."""
    fn = core_lib.lib().aqua_core_inline_round_trip
    fn.argtypes, fn.restype = [ctypes.c_void_p, ctypes.c_uint64, ctypes.c_void_p], ctypes.c_int32
    rng = np.random.default_rng(n)
    d = np.zeros(n, dtype=core_lib.RUN_DESC)
    top = 64 << 30
    d["img_off"] = rng.integers(0, top // 16, n) * 16
    d["img_lstride"] = rng.integers(0, top // 16, n) * 16
    d["block"] = rng.integers(0, 1 << 31, n)
    d["nchunks"] = rng.integers(1, 4097, n)
    if n:
        d["img_off"][0] = d["img_lstride"][-1] = top - 16
    got = np.zeros_like(d)

    def fits(runs):
        return fn(runs.ctypes.data if n else None, n, got.ctypes.data if n else None)

    assert fits(d) == (n <= 224)
    if 0 < n <= 224:
        assert got.tobytes() == d.tobytes()
        for f in ("img_off", "img_lstride"):
            e = d.copy()
            e[f][n // 2] = top
            assert fits(e) == 0


def test_header_states_every_limit_of_runs_in_kernel_arguments():
    """A caller of the allocation-free entry point has to know which of its
    calls use the scratch that pools share: the header names both limits, the
    number of runs and the offset or stride, wherever it names one."""
    fn = core_lib.lib().aqua_core_inline_round_trip
    fn.argtypes, fn.restype = [ctypes.c_void_p, ctypes.c_uint64, ctypes.c_void_p], ctypes.c_int32

    def packs(n, off=0, stride=16):
        d = np.zeros(n, dtype=core_lib.RUN_DESC)
        d["nchunks"], d["img_off"], d["img_lstride"] = 1, off, stride
        got = np.zeros_like(d)
        return fn(d.ctypes.data, n, got.ctypes.data) == 1

    runs = max(n for n in range(1, 1025) if packs(n))
    gib = next(g for g in range(1, 1025) if not packs(1, off=g << 30))
    assert not packs(1, stride=gib << 30) and packs(1, (gib << 30) - 16, (gib << 30) - 16)
    text = open(os.path.join(build.INCLUDE, "aqua.h")).read()
    comment = text[text.index("/* ---- Allocation-free swap"):text.index("aqua_swap_noalloc(")]
    said = " ".join(comment.replace(" * ", " ").split())
    assert said.count(f"at most {runs} runs") == 2, said
    assert said.count(f"{gib} GiB") >= 2, said
    assert f"more than {runs} runs" not in said


@pytest.mark.parametrize("n", [0, 1, 2, 63, 64, 65, 80])
def test_packed_ranges_give_the_planned_pieces(n):
    """The pieces that workgroups find in the packed ranges are those of the
    general plan, in order, empty ranges left out; more than 64 non-empty
    ranges are not packed."""
    L = core_lib.lib()
    U64 = ctypes.c_uint64
    for fn in (L.aqua_core_packed_pieces, L.aqua_core_plan_copies):
        fn.argtypes = [ctypes.c_uint32] + [ctypes.c_void_p] * 4 + [U64]
        fn.restype = ctypes.c_int64
    rng = np.random.default_rng(n)
    sizes = (0, 16, 65520, 65536, 65552, 131072, 1 << 20, 700000 // 16 * 16)
    for trial in range(20):
        ln = rng.choice(sizes, n).astype(np.uint64)
        if trial == 0:
            ln[:] = 65536
        so, do = (rng.integers(0, 1 << 40, n).astype(np.uint64) * 16 for _ in range(2))
        a, b = np.zeros((4096, 4), np.uint64), np.zeros((4096, 4), np.uint64)
        args = (n, so.ctypes.data, do.ctypes.data, ln.ctypes.data)
        got = L.aqua_core_packed_pieces(*args, a.ctypes.data, 4096)
        want = L.aqua_core_plan_copies(*args, b.ctypes.data, 4096)
        if np.count_nonzero(ln) > 64:
            assert got == -1
            continue
        assert got == want <= 4096
        assert np.array_equal(a[:got, :3], b[:got, :3])
        assert np.array_equal(a[:got, 3], np.arange(got, dtype=np.uint64))


@pytest.mark.parametrize("units", [0, 1, 7, 8, 9, 63, 64, 65, 127, 128, 200, 20672])
def test_copy_windows_are_a_bijection(units):
    """Every piece once; within a window of 64 XCD x (= block % 8) takes the
    x-th stretch of adjacent pieces."""
    fn = core_lib.lib().aqua_core_xcd_window_unit
    fn.argtypes, fn.restype = [ctypes.c_uint32] * 2, ctypes.c_uint32
    got = [fn(b, units) for b in range(units)]
    assert sorted(got) == list(range(units))
    for base in range(0, units - 63, 64):
        for x in range(8):
            assert got[base + x:base + 64:8] == list(range(base + 8 * x, base + 8 * x + 8))


def test_link_copies_merge_only_where_both_sides_continue():
    fn = core_lib.lib().aqua_core_append_pieces
    fn.argtypes = [ctypes.c_void_p, ctypes.c_uint64, ctypes.c_void_p]
    fn.restype = ctypes.c_uint64

    def merged(pieces):
        a = np.array(pieces, dtype=np.uint64).reshape(-1, 3)
        out = np.zeros_like(a)
        n = fn(a.ctypes.data, len(a), out.ctypes.data)
        return [tuple(int(x) for x in r) for r in out[:n]]

    assert merged([]) == []
    assert merged([(100, 900, 10), (110, 910, 20), (130, 930, 5)]) == [(100, 900, 35)]
    for apart in ([(100, 900, 10), (110, 911, 20)], [(100, 900, 10), (111, 910, 20)],
                  [(100, 900, 10), (90, 890, 10)], [(100, 900, 10), (100, 900, 10)]):
        assert merged(apart) == apart
    assert merged([(0x100, 0x900, 16), (0x110, 0x910, 16), (0x130, 0x920, 16),
                   (0x140, 0x930, 16)]) == [(0x100, 0x900, 32), (0x130, 0x920, 32)]


def test_ring_space_of_captured_calls_is_never_given_out_again():
    """Random calls over a ring of 64 units, some captured: no call is placed
    over a captured one's space, a call is refused only where no place avoids
    them all, and without captured calls the place is the plain rule's (the
    front if it is free, else behind the last call, else the front)."""
    fn = core_lib.lib().aqua_core_ring_place
    P, U64 = ctypes.c_void_p, ctypes.c_uint64
    fn.argtypes, fn.restype = [U64, U64, U64, P, U64, P, U64], ctypes.c_int64
    rng = np.random.default_rng(5)
    for trial in range(200):
        ring, head, live, kept = 64, 0, [], []
        for _ in range(60):
            n = int(rng.integers(1, 70 if rng.random() < 0.1 else 20))
            la, ka = (np.array(v, dtype=np.uint64).reshape(-1) for v in (live, kept))
            got = fn(ring, n, head, la.ctypes.data, len(live), ka.ctypes.data, len(kept))
            free = [a for a in range(ring - n + 1)
                    if all(h <= a or a + n <= l for l, h in kept)]
            if not free:
                assert got == -1
                continue
            assert got in free
            if not kept:
                front = all(l >= n for l, h in live)
                assert got == (0 if front or head + n > ring else head)
            live = [(l, h) for l, h in live if h <= got or got + n <= l]   # waited for
            live.append((got, got + n))
            head = got + n
            if trial % 2 and rng.random() < 0.1:
                kept.append((got, got + n))
            while live and rng.random() < 0.4:
                live.pop(0)
