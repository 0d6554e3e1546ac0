"""GPU parity of the dense comparator's 256 x 256-tile cache write (enough tokens that the small
tiles would take four rounds of workgroups or more) against the fp64 oracle: two videos of 5,049
tokens, so that a tile spans both and the last one is ragged, and a chunk that wraps the ring.
The widths put the K / V boundary inside a tile (1,280 = 5 tiles of outputs), take heads of 64 and
of 72 channels (heads that straddle waves and tiles), and contract over 2, 6 and 4 LDS stages of
32 columns (fewer than the stages in flight, and more). tests/test_dense_write_rule.py holds the rule
that sends these calls to this kernel. Bars as in tests/test_gpu_dense.py."""
import pytest
import torch

from tests._build_once import ensure_built

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ensure_built()
    import paper_2605_30351_amd as m
    yield m


from tests.gpu_common import host_bits  # noqa: E402
from tests.test_gpu_dense import DenseLayer, check_dense_chunk  # noqa: E402
from workloads import WAN, make_dense_inputs  # noqa: E402


BATCH, GRID_H, GRID_W, CHUNK = 2, 33, 51, 3
SHAPES = [(5, 128, 64), (10, 64, 192), (16, 72, 128)]  # n_heads, d_v, d_model
CU_COUNTS = range(200, 305)  # compute units for which every shape takes this kernel


@pytest.mark.parametrize("n_heads,d_v,d_model", SHAPES)
def test_wide_write(vm, n_heads, d_v, d_model):
    assert torch.cuda.get_device_properties(0).multi_processor_count in CU_COUNTS
    d = WAN.replace(d_model=d_model, n_heads=n_heads, d_v=d_v, grid_h=GRID_H, grid_w=GRID_W,
                    window_frames=5, chunk_frames=CHUNK)
    layer = DenseLayer(vm, make_dense_inputs(d, seed=81, n_frames=6, batch=BATCH))
    for fe in (0, 3):
        before = host_bits(layer.kv)
        layer.write(fe)
        check_dense_chunk(layer, fe, before)
