"""GPU parity of swaps of small chunks: every workgroup width, at chunk sizes
on and beside its edges, against the oracle byte for byte."""
import pytest
import torch

from paper_2407_21255_amd import aqua
from paper_2407_21255_amd import workload as wl
from tests.gpu_util import say
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
def test_every_width_at_its_edges(chunk, long_runs):
    """Single-block runs, and single blocks beside stretches of up to 64 KiB
    whose runs are longer than the mean that sizes the workgroup."""
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
