"""GPU parity of swaps of small chunks and of few runs, against the oracle byte
for byte: chunk sizes on and beside the edges of a wave's 1 KiB and of a row of
1024 lanes; runs in the kernels' arguments, at and beside the number that goes there; and the
descriptor ring, with calls that need it."""
import numpy as np
import pytest
import torch

import oracle
from paper_2407_21255_amd import aqua
from paper_2407_21255_amd import workload as wl
from tests.checkers import assert_bytes_equal
from tests.gpu_util import device_pool, guarded_buffer, host, odesc, say
from tests.test_gpu_swap import _roundtrip

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    aqua.load()
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("long_runs", [False, True], ids=["single", "mixed"])
@pytest.mark.parametrize("chunk", [16, 1008, 1024, 1040, 2048, 2064, 4096, 4112, 6144, 8192,
                                   12288, 16368, 16384])
def test_parts_of_a_run_at_their_edges(chunk, long_runs):
    """Single-block runs, and single blocks beside stretches of up to 64 KiB,
    whose runs have more parts of 1 KiB than the others."""
    shape = wl.KVShape(3, 600, 1, 1, chunk // 2, wl.FP8_E4M3)
    assert shape.chunk_bytes == chunk
    perm = wl.permutation(200, 91)
    scattered = [3 * b for b in perm]              # never consecutive
    if long_runs:
        out_tables = [list(range(100, 160)), [3 * b for b in range(70, 90)], [0]]
        in_tables = [list(range(400, 460)), [3 * b for b in range(160, 180)], [2]]
    else:
        out_tables = [scattered[:37], scattered[37:38], scattered[38:90]]
        in_tables = [scattered[90:127], scattered[127:128], scattered[128:180]]
    say("chunk", chunk, "long runs", long_runs)
    _roundtrip(shape, 91, out_tables, in_tables, None)


@pytest.mark.parametrize("where", ["hbm", "noalloc", "staged", "zero_copy"])
def test_runs_in_kernel_arguments(monkeypatch, where):
    """Calls of 1, 223, 224 and 225 runs, back to back on two streams with no
    host sync: the first three carry their runs in the kernels' arguments.
    Staged calls go through 16 KiB slots, several launches each."""
    monkeypatch.setenv("AQUA_STAGE_SLOT_BYTES", str(16 << 10))
    shape = wl.KVShape(5, 4096, 1, 1, 16, wl.BF16)            # 64-byte chunks
    d = odesc(shape)
    pool = device_pool(shape, 37)
    pool_h = host(pool)
    sizes = [1, 223, 224, 225, 224, 1]
    perm = [2 * b for b in wl.permutation(shape.num_blocks // 2, 37)]   # no two adjoin
    tables, k = [], 0
    for n in sizes:
        tables.append(perm[k:k + n])
        k += n
    fresh = [b + 1 for b in perm[:k]]                          # odd blocks
    G = 4096
    bufs = [guarded_buffer(shape.image_bytes(n), G, where in ("staged", "zero_copy"))
            for n in sizes]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    kv = aqua.KVPool(shape.as_tuple(), pool)
    try:
        kv.set_host_path(aqua.AQUA_HOST_STAGED if where == "staged" else aqua.AQUA_HOST_ZERO_COPY)
        ins, j = [], 0
        for i, (t, buf) in enumerate(zip(tables, bufs)):
            img = buf[G:G + shape.image_bytes(len(t))]
            dst = fresh[j:j + len(t)]
            j += len(t)
            ins.append(dst)
            say(where, "runs", len(t))
            if where == "noalloc":
                kv.swap_noalloc(0, [t], img, stream=streams[i % 2])
                kv.swap_noalloc(1, [dst], img, stream=streams[(i + 1) % 2])
            else:
                kv.swap_out([t], img, stream=streams[i % 2])
                kv.swap_in([dst], img, stream=streams[(i + 1) % 2])
        kv.sync()
        assert kv.stats()["descriptors"] == 2 * sum(sizes)
    finally:
        kv.close()
    for t, dst, buf in zip(tables, ins, bufs):
        want = np.full(buf.numel(), wl.GUARD_BYTE, dtype=np.uint8)
        inner = want[G:G + shape.image_bytes(len(t))]
        assert oracle.swap_out(d, pool_h, [t], inner) == 0
        assert_bytes_equal(host(buf), want, f"image of {len(t)} runs and guards")
        assert oracle.swap_in(d, pool_h, [dst], inner) == 0
    assert_bytes_equal(host(pool), pool_h, "pool")


@pytest.mark.parametrize("where", ["hbm", "staged"])
def test_ring_wraps_under_calls_that_need_it(monkeypatch, where):
    """A 12 KiB ring (384 runs) under calls of 300 runs: each waits for the
    call that used the space last.  Two streams, no host sync."""
    monkeypatch.setenv("AQUA_RING_BYTES", str(12 << 10))
    monkeypatch.setenv("AQUA_STAGE_SLOT_BYTES", str(256 << 10))
    shape = wl.KVShape(2, 8192, 1, 4, 16, wl.BF16)            # 256-byte chunks
    d = odesc(shape)
    pool = device_pool(shape, 41)
    pool_h = host(pool)
    perm = [2 * b for b in wl.permutation(shape.num_blocks // 2, 41)]
    tables = [perm[300 * i:300 * i + 300] for i in range(6)]
    imgs = [guarded_buffer(shape.image_bytes(300), 0, where == "staged") for _ in tables]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    kv = aqua.KVPool(shape.as_tuple(), pool)
    try:
        for i, (t, img) in enumerate(zip(tables, imgs)):
            kv.swap_out([t], img, stream=streams[i % 2])
            kv.swap_in([[b + 1 for b in t]], img, stream=streams[(i + 1) % 2])
        kv.sync()
        say("ring", where, "host wait us", kv.stats()["wait_ns"] // 1000)
    finally:
        kv.close()
    for t, img in zip(tables, imgs):
        want = np.zeros(img.numel(), dtype=np.uint8)
        assert oracle.swap_out(d, pool_h, [t], want) == 0
        assert_bytes_equal(host(img), want, "image")
        assert oracle.swap_in(d, pool_h, [[b + 1 for b in t]], want) == 0
    assert_bytes_equal(host(pool), pool_h, "pool")


@pytest.mark.parametrize("runs", [20, 150, 240])
@pytest.mark.parametrize("entry", ["out", "noalloc"])
def test_one_call_captured_and_replayed(entry, runs):
    """One call captured into a HIP graph (its event is then recorded, not
    carried by the launch), replayed four times over changing pool bytes with
    eager work and a sync in between: every replay equals the gather."""
    shape = wl.KVShape(3, 512, 1, 16, 64, wl.BF16)             # 4 KiB chunks
    pool = device_pool(shape, 43)
    table = [2 * b for b in wl.permutation(shape.num_blocks // 2, 43)[:runs]]
    idx = torch.tensor(table, device="cuda")
    img = torch.zeros(shape.image_bytes(runs), dtype=torch.uint8, device="cuda")
    kv = aqua.KVPool(shape.as_tuple(), pool)

    def call():
        s = torch.cuda.current_stream()
        return kv.swap_out([table], img, stream=s) if entry == "out" else \
            kv.swap_noalloc(0, [table], img, stream=s)

    try:
        call()
        kv.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, capture_error_mode="relaxed"):
            call()
        for k in range(4):
            say(entry, runs, "replay", k)
            img.zero_()
            pool.add_(1)
            graph.replay()
            torch.cuda.synchronize()
            want = pool.view(3, 512, -1)[:, idx].reshape(-1)
            assert torch.equal(img, want), k
    finally:
        kv.close()


@pytest.mark.parametrize("runs", [20, 150, 240])
@pytest.mark.parametrize("entry", ["out", "noalloc"])
def test_replays_between_other_calls_of_the_pool(monkeypatch, entry, runs):
    """Between the replays of a captured call the pool serves eager calls, of
    few runs and of more than travel in arguments, on a ring of 768 runs: they
    take neither the captured call's descriptors nor trouble from its event."""
    monkeypatch.setenv("AQUA_RING_BYTES", str(24 << 10))
    shape = wl.KVShape(3, 1024, 1, 16, 64, wl.BF16)            # 4 KiB chunks
    pool = device_pool(shape, 53)
    perm = [2 * b for b in wl.permutation(shape.num_blocks // 2, 53)]
    table, few, many = perm[:runs], perm[40:60], perm[200:500]
    img, img_few, img_many = (torch.zeros(shape.image_bytes(len(t)), dtype=torch.uint8,
                                          device="cuda") for t in (table, few, many))
    kv = aqua.KVPool(shape.as_tuple(), pool)

    def call(t, dst):
        s = torch.cuda.current_stream()
        return kv.swap_out([t], dst, stream=s) if entry == "out" else \
            kv.swap_noalloc(0, [t], dst, stream=s)

    def gathered(t):
        return pool.view(3, 1024, -1)[:, torch.tensor(t, device="cuda")].reshape(-1)

    try:
        call(many, img_many)
        kv.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, capture_error_mode="relaxed"):
            ticket = call(table, img)
        assert aqua.aqua_query(kv.handle, ticket) == 1   # nothing of it runs yet
        for k in range(4):
            say(entry, runs, "replay", k)
            for _ in range(20):
                call(few, img_few)
                call(many, img_many)
            kv.sync()
            img.zero_()
            pool.add_(1)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(img, gathered(table)), k
            for t, dst in ((few, img_few), (many, img_many)):
                call(t, dst)
                kv.sync()
                assert torch.equal(dst, gathered(t)), k
    finally:
        kv.close()


def test_captured_calls_fill_the_ring(monkeypatch):
    """A ring of 384 runs that a captured call of 240 has taken: a call of 300
    gets new rings, the allocation-free form is refused, and every replay
    still gathers what was captured."""
    monkeypatch.setenv("AQUA_RING_BYTES", str(12 << 10))
    shape = wl.KVShape(3, 1024, 1, 16, 64, wl.BF16)
    pool = device_pool(shape, 59)
    perm = [2 * b for b in wl.permutation(shape.num_blocks // 2, 59)]
    table, many = perm[:240], perm[200:500]
    img, img_many = (torch.zeros(shape.image_bytes(len(t)), dtype=torch.uint8, device="cuda")
                     for t in (table, many))

    def gathered(t):
        return pool.view(3, 1024, -1)[:, torch.tensor(t, device="cuda")].reshape(-1)

    kv = aqua.KVPool(shape.as_tuple(), pool)
    try:
        kv.swap_out([many], img_many)
        kv.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, capture_error_mode="relaxed"):
            kv.swap_out([table], img, stream=torch.cuda.current_stream())
        with pytest.raises(aqua.AquaError) as e:
            kv.swap_noalloc(0, [many], img_many)
        assert e.value.status == aqua.AQUA_ERR_CAPACITY
        for k in range(3):
            say("replay", k)
            img_many.zero_()
            kv.swap_out([many], img_many)                      # the first takes new rings
            kv.sync()
            assert torch.equal(img_many, gathered(many)), k
            img.zero_()
            pool.add_(1)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(img, gathered(table)), k
        kv.swap_noalloc(0, [many], img_many)                   # and they serve it too
        kv.sync()
        assert torch.equal(img_many, gathered(many))
    finally:
        kv.close()


@pytest.mark.parametrize("where", ["hbm", "hbm_capped", "host"])
@pytest.mark.parametrize("n", [1, 9, 64, 65, 130])
def test_range_copies_of_few_and_many_ranges(n, where):
    """Migrations by the range-copy kernel at and beside the number of ranges
    its arguments hold: ragged ranges of 0 bytes to 1.5 MiB, in another order
    at the destination, with gaps that must not change."""
    rng = np.random.default_rng(n)
    sizes = (0, 16, 48, 4096, 65520, 65536, 65552, 200000, 1 << 20, 1500000)
    ln = rng.choice(sizes, n).astype(np.uint64) // 16 * 16
    ln[0] = 327696
    so = np.concatenate([[32], 32 + np.cumsum(ln + 64)[:-1]]).astype(np.uint64)
    total = int((ln + 64).sum()) + 64
    do, at = np.zeros(n, np.uint64), 16
    for k in rng.permutation(n):
        do[k] = at
        at += int(ln[k]) + 32
    src_h = rng.integers(0, 256, total, dtype=np.uint8)
    want = np.full(total, wl.GUARD_BYTE, dtype=np.uint8)
    for s, d, m in zip(so.astype(int), do.astype(int), ln.astype(int)):
        want[d:d + m] = src_h[s:s + m]
    src, dst = torch.from_numpy(src_h), torch.from_numpy(np.full_like(want, wl.GUARD_BYTE))
    src, dst = (src.pin_memory(), dst.pin_memory()) if where == "host" else (src.cuda(), dst.cuda())
    shape = wl.KVShape(2, 16, 1, 2, 8, wl.BF16)
    pool = device_pool(shape, 47)
    kv = aqua.KVPool(shape.as_tuple(), pool)
    try:
        if where == "hbm_capped":
            kv.set_max_workgroups(aqua.AQUA_TARGET_DEVICE, 7)
        say(where, "ranges", n, "bytes", int(ln.sum()))
        kv.migrate(src, dst, so, do, ln)
        kv.sync()
        assert kv.stats()["bytes_migrated"] == int(ln.sum())
    finally:
        kv.close()
    assert_bytes_equal(host(dst), want, "destination and gaps")


def test_default_stream_is_the_current_one():
    """No stream given: the caller's current stream, inside and outside a
    stream context (None stands for the null stream)."""
    assert aqua._stream_handle(None) == (torch.cuda.current_stream().cuda_stream or None)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert aqua._stream_handle(None) == s.cuda_stream
    assert aqua._stream_handle(None) == aqua._stream_handle(torch.cuda.current_stream())
